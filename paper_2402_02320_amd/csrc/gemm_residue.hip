// Exact ring GEMM over Z_2^64 and Z_2^128 on the int8 matrix cores by residues, for products large enough that the
// matrix units bound the digit kernels (gemm_limb.hip, gemm_limb128.hip).
//
// The digit kernels spend ND (ND + 1) / 2 int8 products per ring multiply-add (36 for 8-byte, 136 for 16-byte ring
// elements).  An output element is S mod 2^(8 ND) of the integer S = sum of 2 K products of signed ring elements; S
// is determined by its residues modulo L pairwise coprime moduli of eight bits whose product exceeds 2 |S|
// (residue_tables.hpp): L = 18 (36) int8 products per multiply-add, every modulus an ordinary int8 GEMM with int32
// accumulation.  All steps are exact integer arithmetic, so the words are those of the digit kernels.
//
//  residue_pack_kernel     opens E (F), converts E, A_i (F, B_i') to balanced digits and these to L residues, one
//                          signed byte each, laid out as fragments of v_mfma_i32_16x16x64_i8; right operands carry
//                          the factor (P/p_l)^-1 of the reconstruction.
//  residue_gemm_kernel     Y_l = [E | A_i] . [B_i' ; F] mod p_l, one byte per element and modulus.
//  residue_combine_kernel  S from the L bytes of an element, Z_i = C_i + S.
//
// Measured, whole call, digit kernels against this: 5 parties 4096^3 17.6 -> 10.9 ms (GEMM 8.8, pack 1.5, combine 0.6 ms),
// 2 x 2048^3 over Z_2^128 3.4 -> 1.33 ms.  The GEMM runs at 0.55 to 0.57 of the nominal int8 peak, 0.80 of what a register-only
// loop sustains on random bytes; without its loads it would be 14 % faster (10 % of that are L2 misses), without its
// epilogue 2 %.  The matrix pipes are busy 0.71 of the cycles at 1.9 GHz, the L2 0.95 of them (11.4 TB/s, hit rate 0.80): it is
// bound by the power of matrix units and operand traffic together; a fifth LDS stage, another order of the two operand
// pairs on half of the XCDs, or loads bunched in the first half of a step change it by 1 %.
//
// Fragment: 16 rows (columns) x 64 k = 1 KiB; lane l's 16 bytes at 16 l are row l % 16, k = 16 (l / 16) + 0..15.
// Store of one operand: [modulus][panel of 256 rows][kt64][16 fragments][1024], so that a workgroup's share of one
// k-step is 16 KiB in a row.
#include <algorithm>

#include "limb_common.hpp"
#include "residue_tables.hpp"

namespace spin {
namespace {

constexpr int kPanel = 256;                              // rows (columns) of an operand panel and of an output tile
constexpr int kStepK = 64;                               // inner dimension of one k-step
constexpr int kPanelStep = kPanel * kStepK;              // bytes of one panel's k-step

// ------------------------------------------------------------------ pack ---
template <class T> struct ResidueSide {
    const T *val, *tri;       // X, A or Y, B of this batch entry (party 0)
    size_t party_stride;      // elements between two parties' matrices
    int rows, cols;           // source matrix, row-major
    int line0;                // first row (left, transposed right) or column (right) of the panels
    int k0, k1;               // inner dimension range
    char *opened, *triple;    // fragment stores: the opened matrix; one slot per party of [first, last)
    int first, last;          // parties whose triple share is converted
    int open;                 // whether the opened matrix is formed and converted (party 0 of a right side needs it)
    int panels, KT;
};
template <class T> struct ResiduePackArgs {
    ResidueSide<T> left, right;
    int n;
    unsigned left_blocks;
};

// Consecutive k that one lane converts: 128 bytes of source in registers.
template <class T> constexpr int kPackRun = 128 / sizeof(T);

// EL consecutive k of one row (column) as balanced digits -> L residues of EL bytes, modulus l at dst (a scalar) +
// l * mod_stride + lane_at.
// Per element and modulus: the weighted digit sum (a 4-byte dot product per word), the remainder through a
// reciprocal, and a quarter of the byte merge -- about six vector instructions.  They mostly hide behind the memory traffic
// (8 bytes in, 18 out): leaving all of them out changes the packs of five parties 4096^3 from 1.51 to 1.40 ms a call (one party at a
// time; in two blocks of all parties from 1.32 to 1.27), of two parties 2048^3 over Z_2^128 from 317 to 286 us.
// Stores are 16 bytes per lane, whole 256-byte runs per 16 lanes.  With 16-byte ring elements a lane converts only 8 k
// (128 bytes of source in registers); lanes l and l + 32 hold the two halves of a 16-byte run and trade them between
// two moduli, the lower lanes storing the even, the upper lanes the odd one.
template <class T, bool RIGHT, int EL> __device__ __forceinline__ void store_residues(const T (&digits)[EL], char *dst, u32 lane_at, size_t mod_stride)
{
    constexpr int L = ResidueTables<T>::L, NW = ResidueTables<T>::NW;
    static_assert(EL == 16 || (EL == 8 && L % 2 == 0), "a lane stores 16 bytes");
    if (EL == 8) dst += threadIdx.x % 64 / 32 * mod_stride;
    u32 even[EL / 4];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        u32 x[EL], row[EL / 4];
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            int sum = (int)kResidue<T>.offset[l];
#pragma unroll
            for (int w = 0; w < NW; ++w)
                sum = __builtin_amdgcn_sdot4((int)(u32)(digits[e] >> (32 * w)),
                                             (int)(RIGHT ? kResidue<T>.right[l][w] : kResidue<T>.left[l][w]), sum, false);
            x[e] = (u32)sum;
        }
#pragma unroll
        for (int e = 0; e < EL; ++e) x[e] -= (u32)__mul24((int)__umulhi(x[e], kResidue<T>.recip[l]), kModuli[l]);
#pragma unroll
        for (int q = 0; q < EL / 4; ++q) {
            // the remainders carry an offset of 128: as signed bytes they are the residues once the top bit is flipped
            const u32 lo = __builtin_amdgcn_perm(x[4 * q + 1], x[4 * q], 0x0c0c0400u);
            const u32 hi = __builtin_amdgcn_perm(x[4 * q + 3], x[4 * q + 2], 0x04000c0cu);
            row[q] = (lo | hi) ^ 0x80808080u;
        }
        if constexpr (EL == 16) {
            *(v4i *)(dst + lane_at) = v4i{(int)row[0], (int)row[1], (int)row[2], (int)row[3]};
            dst += mod_stride;
        } else if (l % 2 == 0) {
#pragma unroll
            for (int q = 0; q < EL / 4; ++q) even[q] = row[q];
        } else {
            const auto s0 = __builtin_amdgcn_permlane32_swap(even[0], row[0], false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(even[1], row[1], false, false);
            *(v4i *)(dst + lane_at) = v4i{(int)s0[0], (int)s1[0], (int)s0[1], (int)s1[1]};
            dst += 2 * mod_stride;
        }
        __builtin_amdgcn_sched_barrier(0);               // one modulus at a time: interleaved they take 50 registers more
    }
}

// A matrix whose rows are fragment rows (left operands, transposed right operands): a wave reads its 16 x 64 tile as
// row segments (16 bytes per lane), sums the parties' shares in that layout and turns each tile through LDS.
template <class T, bool VEC, bool RIGHT, int WAVES>
__device__ __forceinline__ void residue_pack_rows(const ResidueSide<T> &a, int n, unsigned block, char *lds)
{
    constexpr int ND = sizeof(T);
    constexpr int EL = kPackRun<T>, kSpan = 4 * EL, kParts = kStepK / kSpan;           // k of a lane, of a wave
    constexpr int EPL = 16 / ND, LPR = kSpan / EPL, RPL = 64 / LPR, NL = 16 / RPL;      // u64: 2, 32, 2, 8; u128: 1, 32, 2, 8
    constexpr int kRowBytes = kSpan * ND + 16;
    struct alignas(16) Pair { T e[EPL]; };
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const long tile = (long)block * WAVES + wave;        // (panel, kt, part of the k-step, fragment)
    if (tile >= (long)a.panels * a.KT * (16 * kParts)) return;   // whole waves leave; each works in its own part of LDS
    const int frag = (int)(tile % 16), part = (int)(tile / 16 % kParts);
    const long pk = tile / (16 * kParts);
    const int kt = (int)(pk % a.KT), panel = (int)(pk / a.KT);
    const int row0 = a.line0 + panel * kPanel + frag * 16, kk = a.k0 + kt * kStepK + part * kSpan + EPL * (lane % LPR);
    const size_t mod_stride = (size_t)a.panels * a.KT * kPanelStep;
    const size_t slot = mod_stride * ResidueTables<T>::L;
    // this lane's run of k in the wave's span: 16 (lane / 16), or, with runs of 8, 16 ((lane / 16) % 2) + 8 (lane / 32)
    const int run = EL == 16 ? 16 * (lane / 16) : lane / 16 % 2 * 16 + lane / 32 * 8;
    const size_t at = (size_t)pk * kPanelStep + frag * 1024;
    const u32 lane_at = (part * kSpan + run) / 16 * 256 + (lane % 16) * 16;
    // Loads are unconditional and nothing is masked on the way in: an element outside the matrix reads one inside.
    // Rows beyond the matrix only reach outputs that are never stored, and for k >= k1 the right operand's digits are
    // zeroed before the conversion.  The tile's first row is a scalar base, a lane's place in it a 32-bit offset (16
    // rows of at most 2^24 elements of 16 bytes).
    const int base_row = min(row0, a.rows - 1);
    const size_t base = (size_t)base_row * a.cols;
    u32 off[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j)
        off[j] = ((u32)(min(row0 + RPL * j + lane / LPR, a.rows - 1) - base_row) * (u32)a.cols + (u32)min(kk, a.k1 - (VEC ? EPL : 1))) * ND;
    auto load = [&](const T *matrix, Pair (&v)[NL]) {
        const char *src = (const char *)(matrix + base);
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            if (VEC) {
                v[j] = *(const Pair *)(src + off[j]);
            } else {
#pragma unroll
                for (int q = 0; q < EPL; ++q) v[j].e[q] = *(const T *)(src + (off[j] + (kk + q < a.k1 ? q * ND : 0)));
            }
        }
    };
    char *mine = lds + wave * 16 * kRowBytes;
    auto turn_and_store = [&](const Pair (&v)[NL], char *dst) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the previous round's reads are done (one wave, in order)
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            Pair d;
#pragma unroll
            for (int q = 0; q < EPL; ++q) d.e[q] = RIGHT && kk + q >= a.k1 ? (T)0 : to_digits<T>(v[j].e[q]);
            *(Pair *)(mine + (RPL * j + lane / LPR) * kRowBytes + (lane % LPR) * 16) = d;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        T w[EL];
#pragma unroll
        for (int j = 0; j < EL / EPL; ++j) {
            const Pair d = *(const Pair *)(mine + (lane % 16) * kRowBytes + run * ND + j * 16);
#pragma unroll
            for (int q = 0; q < EPL; ++q) w[EPL * j + q] = d.e[q];
        }
        store_residues<T, RIGHT>(w, dst + at, lane_at, mod_stride);
    };
    // One conversion in the code for all slots: pass i < n brings party i's triple share (and adds it to the opened
    // matrix), pass n the opened matrix, pass n + 1 of a right side B_0 + F, party 0's slot.
    Pair opened[NL], tv[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
        for (int q = 0; q < EPL; ++q) opened[j].e[q] = 0;
    const int end = a.open ? n + (RIGHT && a.first == 0 ? 2 : 1) : a.last;
    for (int i = a.open ? 0 : a.first; i < end; ++i) {
        char *dst = i < n ? a.triple + (size_t)(i - a.first) * slot : i == n ? a.opened : a.triple;
        if (i != n) load(a.tri + (i < n ? i : 0) * a.party_stride, tv);
        if (i < n && a.open) {
            Pair xv[NL];
            load(a.val + i * a.party_stride, xv);
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int q = 0; q < EPL; ++q) opened[j].e[q] += xv[j].e[q] - tv[j].e[q];
            if (i < a.first || i >= a.last || (RIGHT && i == 0)) continue;
        }
        if (i >= n) {
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int q = 0; q < EPL; ++q) tv[j].e[q] = opened[j].e[q] + (i == n ? (T)0 : tv[j].e[q]);
        }
        turn_and_store(tv, dst);
    }
}

// A right operand stored K x N: a wave takes 64 columns x 16 k of a k-step, or, with runs of 8, 32 columns x 16 k (the
// lower lanes the first 8), so that every load covers whole 512-byte row segments.
template <class T, int WAVES>
__device__ __forceinline__ void residue_pack_columns(const ResidueSide<T> &a, int n, unsigned block)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    constexpr int EL = kPackRun<T>, kCols = EL == 16 ? 64 : 32, kGroups = kPanel / kCols;
    const long tile = (long)block * WAVES + wave;        // (panel, kt, quarter of the k-step, group of columns)
    if (tile >= (long)a.panels * a.KT * (4 * kGroups)) return;
    const int group = (int)(tile % kGroups), quarter = (int)(tile / kGroups % 4);
    const long pk = tile / (4 * kGroups);
    const int kt = (int)(pk % a.KT), panel = (int)(pk / a.KT);
    const int col0 = a.line0 + panel * kPanel + group * kCols, col = col0 + lane % kCols;
    const int kk0 = a.k0 + kt * kStepK + quarter * 16, kk = kk0 + lane / kCols * EL;
    const size_t mod_stride = (size_t)a.panels * a.KT * kPanelStep;
    const size_t slot = mod_stride * ResidueTables<T>::L;
    const size_t at = (size_t)pk * kPanelStep + group * (kCols / 16 * 1024) + quarter * 256;
    const u32 lane_at = lane % kCols / 16 * 1024 + lane % 16 * 16;
    const int base_row = min(kk0, a.k1 - 1), base_col = min(col0, a.cols - 1);   // scalars; unmasked loads as above
    const size_t base = (size_t)base_row * a.cols + base_col;
    const u32 lane_off = (u32)(min(col, a.cols - 1) - base_col) * sizeof(T);
    auto load = [&](const T *matrix, T (&v)[EL]) {
        const char *src = (const char *)(matrix + base);
#pragma unroll
        for (int j = 0; j < EL; ++j)
            v[j] = *(const T *)(src + (lane_off + (u32)(min(kk + j, a.k1 - 1) - base_row) * (u32)a.cols * (u32)sizeof(T)));
    };
    auto store = [&](const T (&v)[EL], char *dst) {
        T d[EL];
#pragma unroll
        for (int j = 0; j < EL; ++j) d[j] = kk + j >= a.k1 ? (T)0 : to_digits<T>(v[j]);
        store_residues<T, true>(d, dst + at, lane_at, mod_stride);
    };
    T opened[EL], tv[EL];
#pragma unroll
    for (int j = 0; j < EL; ++j) opened[j] = 0;
    const int end = a.open ? n + (a.first == 0 ? 2 : 1) : a.last;
    for (int i = a.open ? 0 : a.first; i < end; ++i) {   // passes as in residue_pack_rows
        char *dst = i < n ? a.triple + (size_t)(i - a.first) * slot : i == n ? a.opened : a.triple;
        if (i != n) load(a.tri + (i < n ? i : 0) * a.party_stride, tv);
        if (i < n && a.open) {
            T xv[EL];
            load(a.val + i * a.party_stride, xv);
#pragma unroll
            for (int j = 0; j < EL; ++j) opened[j] += xv[j] - tv[j];
            if (i < a.first || i >= a.last || i == 0) continue;
        }
        if (i >= n) {
#pragma unroll
            for (int j = 0; j < EL; ++j) tv[j] = opened[j] + (i == n ? (T)0 : tv[j]);
        }
        store(tv, dst);
    }
}

template <class T> constexpr int kPackWaves = 4;
template <class T> inline unsigned residue_pack_blocks(int panels, int KT)
{
    return (unsigned)(((long)panels * KT * (256 / kPackRun<T>) + kPackWaves<T> - 1) / kPackWaves<T>);
}

// Both sides in one launch: the first left_blocks workgroups convert the left operands, the others the right ones.
template <class T, bool VEC, bool TRANSPOSED>
__global__ __launch_bounds__(64 * kPackWaves<T>, 2) void residue_pack_kernel(ResiduePackArgs<T> a)
{
    __shared__ __attribute__((aligned(16))) char lds[kPackWaves<T> * 16 * (4 * kPackRun<T> * sizeof(T) + 16)];
    if (blockIdx.x < a.left_blocks) residue_pack_rows<T, VEC, false, kPackWaves<T>>(a.left, a.n, blockIdx.x, lds);
    else if (TRANSPOSED) residue_pack_rows<T, VEC, true, kPackWaves<T>>(a.right, a.n, blockIdx.x - a.left_blocks, lds);
    else residue_pack_columns<T, kPackWaves<T>>(a.right, a.n, blockIdx.x - a.left_blocks);
}

// ------------------------------------------------------------------ GEMM ---
struct ResidueGemmArgs {
    const char *E, *A, *F, *B;       // fragment stores; A, B: one slot per party of this launch
    size_t a_slot, b_slot;           // bytes of a slot
    size_t a_mod, b_mod;             // bytes of one modulus of a slot
    char *y;                         // [party][modulus][tile][wave][chunk][1024]
    int parties, L, tilesM, tilesN, KT;
    unsigned first_item, items;      // modulus x party x tile: this launch takes [first_item, first_item + items)
    unsigned whole;                  // of them, those in whole rounds of the grid; the rest are shared, `parts` workgroups each
    int parts;
    char *y_parts;                   // residues of the later parts: [item - whole][part - 1][tile]
};

// Persistent: one workgroup per CU, items dealt in rounds so that the 32 workgroups of an XCD work on neighbouring
// tiles of one modulus.  4 waves as 2 x 2, wave tile 128 x 16 NJ = 8 x NJ MFMA tiles of 16 x 16.  The k-steps of all
// items form one sequence through a ring of four LDS stages: in iteration s the wave runs the 8 NJ MFMAs of step s on
// registers, reads the 8 + NJ fragments of step s + 1 into the other register buffer and issues its share of the
// loads of step s + 4 into the stage that step s has left.  The loads run ahead across item boundaries, so the next
// item's first steps are in LDS while the accumulators of this one are reduced and stored.  Past the last item the
// load cursor stands still and refetches its last step, which nothing uses.
constexpr int kMaxRounds = 2048;                         // items of one workgroup in a launch

template <int NJ> struct ResidueShape {
    static constexpr int NSTAGE = 4;
    static constexpr int ahead = NSTAGE - 2;             // whole steps that stay in flight over a wait
    static constexpr int BN = 2 * 16 * NJ;
    static constexpr int a_bytes = kPanelStep, b_bytes = BN * kStepK, stage_bytes = a_bytes + b_bytes;
    static constexpr int lds_bytes = NSTAGE * stage_bytes + kMaxRounds * 16;
    static constexpr int a_loads = 4, b_loads = NJ / 2, loads = a_loads + b_loads;     // per wave and step
    static constexpr int frags = 8 + NJ;                 // LDS -> register reads per wave and step
    static constexpr int stores = 2 * NJ;                // epilogue stores of a wave (16 bytes per lane)
    static constexpr int tile_bytes = kPanel * BN;
};

template <class T, int NJ>
__global__ __launch_bounds__(256) void residue_gemm_kernel(ResidueGemmArgs g)
{
    using S = ResidueShape<NJ>;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wm = wave / 2, wn = wave % 2;
    const u32 lane16 = lane * 16;
    const unsigned tiles = (unsigned)(g.tilesM * g.tilesN);
    // Workgroup ids are dealt round-robin to the XCDs: workgroup w takes item (w % 8) (grid / 8) + w / 8 of each round
    // of gridDim.x items.  Where an item's operands and results lie is worked out for all rounds at once, one round a
    // thread, and kept in LDS behind the stages: half a dozen integer divisions per item would otherwise sit between
    // the matrix instructions (about 300 scalar instructions).
    const unsigned first = gridDim.x % 8 == 0 ? blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8 : blockIdx.x;
    // The items beyond the last whole round would leave most of the grid idle: each is shared by `parts` workgroups, which
    // take an even-length run of its k-steps each (the same run of neighbouring tiles on neighbouring workgroups).
    const unsigned rest = g.items - g.whole;
    const int part = rest > 0 ? (int)(first / rest) : g.parts;           // >= parts: nothing of the rest
    const bool shares = part < g.parts;
    const int rounds = (int)(g.whole / gridDim.x) + (shares ? 1 : 0);    // at most kMaxRounds: the host splits the launch
    if (rounds == 0) return;                             // whole workgroup
    const int part_s0 = shares ? 2 * (part * g.KT / g.parts) : 0, part_s1 = shares ? 2 * ((part + 1) * g.KT / g.parts) : 0;
    v4i *table = (v4i *)(lds + S::NSTAGE * S::stage_bytes);
    for (int r = threadIdx.x; r < rounds; r += 256) {
        const bool shared_item = shares && r == rounds - 1;
        const unsigned local = shared_item ? g.whole + first % rest : first + (unsigned)r * gridDim.x;
        const unsigned id = g.first_item + local, pm = id / tiles, tile = id % tiles;
        const unsigned party = pm % (unsigned)g.parties, mod = pm / (unsigned)g.parties;
        const TileId t = tile_of(tile, g.tilesM, g.tilesN);
        constexpr int per_panel = kPanel / S::BN;        // output tiles to a panel of columns
        v4i e;
        e.x = (int)((mod * g.a_mod + (size_t)t.tm * g.KT * kPanelStep) >> 10);
        e.y = (int)((mod * g.b_mod + (size_t)(t.tn / per_panel) * g.KT * kPanelStep + (t.tn % per_panel) * S::b_bytes) >> 10);
        // later parts lie behind all first ones (negative: counted from y_parts)
        e.z = shared_item && part > 0 ? ~(int)((local - g.whole) * (g.parts - 1) + part - 1) : (int)((party * g.L + mod) * tiles + tile);
        e.w = (int)(mod | party << 16);
        table[r] = e;
    }
    __syncthreads();
    struct Item { u32 a_kb, b_kb; int y_tile, mod, party; };             // fragment offsets in KiB
    auto item_of = [&](int r) {
        const v4i e = table[r];
        Item i;
        i.a_kb = (u32)__builtin_amdgcn_readfirstlane(e.x);
        i.b_kb = (u32)__builtin_amdgcn_readfirstlane(e.y);
        i.y_tile = __builtin_amdgcn_readfirstlane(e.z);
        const int w = __builtin_amdgcn_readfirstlane(e.w);
        i.mod = w & 0xffff;
        i.party = w >> 16;
        return i;
    };

    // ---- load cursor
    const u32 lds0 = (u32)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const size_t wave_a = wave * (S::a_loads * 1024), wave_b = wave * (S::b_loads * 1024);
    int ld_round = 0;
    Item ld;
    const char *ld_a, *ld_b;
    int ld_left, ld_second;                              // steps left in this operand pair, and then in the second one
    auto at_kb = [](const char *base, u32 kb) { return base + ((size_t)kb << 10); };
    auto first_pair = [&](int kt) {                      // (E, B_i') from k-step kt on
        ld_a = at_kb(g.E, ld.a_kb) + wave_a + (size_t)kt * kPanelStep;
        ld_b = at_kb(g.B, ld.b_kb) + ld.party * g.b_slot + wave_b + (size_t)kt * kPanelStep;
    };
    auto second_pair = [&](int kt) {                     // (A_i, F)
        ld_a = at_kb(g.A, ld.a_kb) + ld.party * g.a_slot + wave_a + (size_t)kt * kPanelStep;
        ld_b = at_kb(g.F, ld.b_kb) + wave_b + (size_t)kt * kPanelStep;
    };
    auto set_item = [&]() {
        ld = item_of(ld_round);
        const bool shared_item = shares && ld_round == rounds - 1;
        const int s0 = shared_item ? part_s0 : 0, s1 = shared_item ? part_s1 : 2 * g.KT;
        if (s0 < g.KT) {
            first_pair(s0);
            ld_left = min(s1, g.KT) - s0;
            ld_second = max(s1 - g.KT, 0);
        } else {
            second_pair(s0 - g.KT);
            ld_left = s1 - s0;
            ld_second = 0;
        }
    };
    set_item();
    size_t ld_inc = kPanelStep;
    u32 ld_stage = 0;
    auto issue_load = [&](int q) {                       // q is a constant after unrolling
        if (q < S::a_loads) load_fragment_to_lds(ld_a + q * 1024, lds0 + ld_stage + (u32)wave_a + q * 1024, lane16);
        else load_fragment_to_lds(ld_b + (q - S::a_loads) * 1024,
                                  lds0 + ld_stage + S::a_bytes + (u32)wave_b + (q - S::a_loads) * 1024, lane16);
    };
    auto advance_load_cursor = [&]() {
        ld_stage = ld_stage == (S::NSTAGE - 1) * S::stage_bytes ? 0 : ld_stage + S::stage_bytes;
        if (--ld_left != 0) {
            ld_a += ld_inc;
            ld_b += ld_inc;
        } else if (ld_second > 0) {
            ld_left = ld_second;
            ld_second = 0;
            second_pair(0);
        } else if (ld_round + 1 < rounds) {
            ++ld_round;
            set_item();
        } else {
            ld_inc = 0;                                  // nothing is left: stand still
            ld_left = 0x7fffffff;
        }
    };

    // ---- read cursor
    // Scalars with the stage in them, the lane's place added at the load: as lane addresses beside a stage they took two registers
    // more than there are, spilled around every item.
    const u32 rd_a0 = wm * 8192, rd_b0 = S::a_bytes + wn * (NJ * 1024);
    u32 rd_a = rd_a0, rd_b = rd_b0;
    v4i fr[2][S::frags];                                 // [NJ right fragments, 8 left fragments]
    auto read_fragment = [&](int q) -> v4i {
        return *(const v4i *)(lds + (q < NJ ? rd_b : rd_a) + lane16 + (q < NJ ? q : q - NJ) * 1024);
    };
    auto advance_read_cursor = [&]() {
        const bool last = rd_a == rd_a0 + (S::NSTAGE - 1) * S::stage_bytes;
        rd_a = last ? rd_a0 : rd_a + S::stage_bytes;
        rd_b = last ? rd_b0 : rd_b + S::stage_bytes;
    };

    v4i acc[8][NJ];
    int fresh = 0;                                       // iterations whose wait has the epilogue's stores among the younger accesses

#pragma unroll
    for (int s = 0; s < S::NSTAGE; ++s) {
#pragma unroll
        for (int q = 0; q < S::loads; ++q) issue_load(q);
        advance_load_cursor();
    }
    wait_loads<(S::NSTAGE - 1) * S::loads>();
    workgroup_barrier();
#pragma unroll
    for (int q = 0; q < S::frags; ++q) fr[0][q] = read_fragment(q);
    advance_read_cursor();

    auto iteration = [&](auto cur_c, auto first_c) {
        constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
        constexpr bool FIRST = decltype(first_c)::value;
        // steps s+1 .. s+NSTAGE-1 are in flight, in order: wait for s+1
        if (fresh > 0) { wait_loads<S::ahead * S::loads + S::stores>(); --fresh; }
        else wait_loads<S::ahead * S::loads>();
        wait_lds();                                      // this step's fragments are in registers
        workgroup_barrier();
        int slot = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fr[cur][NJ + i], fr[cur][j], FIRST ? (v4i)(0) : acc[i][j], 0, 0, 0);
                constexpr int total = 8 * NJ;
                constexpr int rd_every = total * 3 / 4 / S::frags;           // 3 (NJ = 8), 2 (NJ = 4)
                constexpr int ld_every = (total - 4) / S::loads;             // 7, 4
                if (slot % rd_every == 0 && slot / rd_every < S::frags) {
                    fr[nxt][slot / rd_every] = read_fragment(slot / rd_every);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (slot % ld_every == 2 && slot / ld_every < S::loads) {
                    issue_load(slot / ld_every);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (slot == total - 4) {
                    advance_read_cursor();
                    advance_load_cursor();
                    __builtin_amdgcn_sched_barrier(0);
                }
                ++slot;
            }
    };
    using Y = std::true_type;
    using N = std::false_type;
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    for (int round = 0; round < rounds; ++round) {
        const int steps = shares && round == rounds - 1 ? part_s1 - part_s0 : 2 * g.KT;      // even
        iteration(B0(), Y());
        iteration(B1(), N());
        for (int s = 2; s < steps; s += 2) {
            iteration(B0(), N());
            iteration(B1(), N());
        }
        // acc mod p, one byte each: q = floor(acc / p) exactly up to a wrap of the remainder to p itself
        const Item it = item_of(round);
        const int p = kModuli[it.mod], recip = kResidue<T>.acc_recip[it.mod], shift = kResidue<T>.acc_shift[it.mod];
        char *dst = (it.y_tile >= 0 ? g.y + (size_t)it.y_tile * S::tile_bytes : g.y_parts + (size_t)~it.y_tile * S::tile_bytes) +
                    wave * (S::stores * 1024) + lane16;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int jq = 0; jq < NJ / 4; ++jq) {
                v4i out;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    int x[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int v = acc[i][4 * jq + j][r];
                        x[r] = v - __mul24(__mulhi(v, recip) >> shift, p);
                    }
                    const u32 lo = __builtin_amdgcn_perm((u32)x[1], (u32)x[0], 0x0c0c0400u);
                    const u32 hi = __builtin_amdgcn_perm((u32)x[3], (u32)x[2], 0x04000c0cu);
                    out[j] = (int)(lo | hi);
                }
                *(v4i *)(dst + (i * (NJ / 4) + jq) * 1024) = out;
            }
        fresh = S::NSTAGE - 1;
    }
    wait_loads<0>();                                     // no load may land after the workgroup's LDS is given back
}

// --------------------------------------------------------------- combine ---
template <class T> struct ResidueCombineArgs {
    const char *y;                   // [party][modulus][tile][wave][chunk][1024], as the GEMM left it
    const T *C;                      // party 0's matrix of this batch entry, and so on
    T *Z;
    size_t party_stride;             // elements between two parties' matrices
    int M, N, row0, col0;            // whole output; first row and column of this block of tiles
    int tilesM, tilesN, parties;
    unsigned waves;                  // parties x tiles x 4 x chunks
    const char *y_parts;             // residues of the items from `whole` on that came in `parts` parts, the later ones
    unsigned whole;
    int parts;
};

// (a + b) mod p of four bytes each, up to a multiple of p that leaves it a byte: both are at most p, and a sum of p or more
// loses p.
__device__ inline u32 add_residues(u32 a, u32 b, u32 p)
{
    const u32 pp = p | p << 16;
    u32 r[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32 sum = ((a >> (8 * h)) & 0x00ff00ffu) + ((b >> (8 * h)) & 0x00ff00ffu);     // below 2^10 each
        const u32 test = sum + (0x02000200u - pp);       // bit 9 of a half: sum >= p
        const u32 mask = ((test >> 9) & 0x00010001u) * 0xffffu;
        r[h] = sum - (pp & mask);
    }
    return r[0] | r[1] << 8;
}

// One lane: the 16 bytes per modulus that one lane of the GEMM stored = 4 rows x 4 columns (16 apart).  S of an
// element is a sum of byte products: with y_l and the bytes of P/p_l as operands of 4-byte dot products, byte column j
// of the result costs a fourth of L instructions; Q joins as one more factor with the bytes of -P.
template <class T, int NJ, bool PARTS>
__global__ __launch_bounds__(256) void residue_combine_kernel(ResidueCombineArgs<T> a)
{
    using S = ResidueShape<NJ>;
    using R = ResidueTables<T>;
    const unsigned w = blockIdx.x * 4 + threadIdx.x / 64;
    if (w >= a.waves) return;
    const int lane = threadIdx.x % 64;
    const unsigned chunk = w % S::stores, wave = w / S::stores % 4, pt = w / S::stores / 4;
    const unsigned tiles = (unsigned)(a.tilesM * a.tilesN), party = pt / tiles, tile = pt % tiles;
    const char *src = a.y + ((size_t)party * R::L * tiles + tile) * S::tile_bytes + (wave * S::stores + chunk) * 1024 + lane * 16;
    const size_t mod_stride = (size_t)tiles * S::tile_bytes;
    v4i y[R::L];
#pragma unroll
    for (int l = 0; l < R::L; ++l) y[l] = *(const v4i *)(src + l * mod_stride);
    // Later parts are fetched six moduli at a time, so that their loads fly together; a modulus whose item is whole
    // fetches its own residues again and adds zero.
    if constexpr (PARTS) {
        const size_t in_tile = (wave * S::stores + chunk) * 1024 + lane * 16;
        auto item = [&](int l) { return (l * (unsigned)a.parties + party) * tiles + tile; };     // the GEMM's numbering
        constexpr int kTogether = 6;
        static_assert(R::L % kTogether == 0, "whole groups of moduli");
#pragma unroll
        for (int l0 = 0; l0 < R::L; l0 += kTogether) {
            if (item(l0 + kTogether - 1) < a.whole) continue;            // items of later moduli have higher numbers
            for (int part = 1; part < a.parts; ++part) {
                v4i more[kTogether];
#pragma unroll
                for (int k = 0; k < kTogether; ++k) {
                    const unsigned id = item(l0 + k);
                    const char *from = id < a.whole ? src + (l0 + k) * mod_stride
                                                    : a.y_parts + (size_t)((id - a.whole) * (a.parts - 1) + part - 1) * S::tile_bytes + in_tile;
                    more[k] = *(const v4i *)from;
                }
#pragma unroll
                for (int k = 0; k < kTogether; ++k) {
                    const u32 mask = item(l0 + k) < a.whole ? 0u : ~0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        y[l0 + k][j] = (int)add_residues((u32)y[l0 + k][j], (u32)more[k][j] & mask, kModuli[l0 + k]);
                }
            }
        }
    }

    const TileId t = tile_of(tile, a.tilesM, a.tilesN);
    const int row = a.row0 + t.tm * kPanel + (int)(wave / 2) * 128 + (int)(chunk / (NJ / 4)) * 16 + 4 * (lane / 16);
    const int col = a.col0 + t.tn * S::BN + (int)(wave % 2) * (16 * NJ) + (int)(chunk % (NJ / 4)) * 64 + lane % 16;
    const T *Cp = a.C + party * a.party_stride;
    T *Zp = a.Z + party * a.party_stride;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        T c[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)                      // rows and columns beyond the matrix are redirected, never stored
            c[r] = Cp[(size_t)min(row + r, a.M - 1) * a.N + min(col + 16 * j, a.N - 1)];
        u32 yq[4][R::groups];                            // [row][group of four moduli]
#pragma unroll
        for (int q = 0; q < R::groups; ++q) {
            const u32 w0 = (u32)y[4 * q < R::L ? 4 * q : 0][j], w1 = (u32)y[4 * q + 1 < R::L ? 4 * q + 1 : 0][j];
            const u32 w2 = 4 * q + 2 < R::L ? (u32)y[4 * q + 2 < R::L ? 4 * q + 2 : 0][j] : 0;
            const u32 w3 = 4 * q + 3 < R::L ? (u32)y[4 * q + 3 < R::L ? 4 * q + 3 : 0][j] : 0;
            if (4 * q >= R::L) {                         // the group of Q alone
#pragma unroll
                for (int r = 0; r < 4; ++r) yq[r][q] = 0;
                continue;
            }
            const u32 t0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), t1 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
            const u32 t2 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), t3 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
            yq[0][q] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
            yq[1][q] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
            yq[2][q] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
            yq[3][q] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            u32 frac = R::two_level ? 0 : 1u << (R::frac_bits - 1);
#pragma unroll
            for (int q = 0; q < R::groups; ++q) frac = __builtin_amdgcn_udot4(yq[r][q], kResidue<T>.frac_hi[q], frac, false);
            if constexpr (R::two_level) {
                frac = (frac << 8) + (1u << (R::frac_bits - 1));
#pragma unroll
                for (int q = 0; q < R::groups; ++q) frac = __builtin_amdgcn_udot4(yq[r][q], kResidue<T>.frac_lo[q], frac, false);
            }
            yq[r][R::L / 4] |= (frac >> R::frac_bits) << (8 * (R::L % 4));       // Q <= L + 1
            T sum = c[r];
#pragma unroll
            for (int word = 0; word < R::NW; ++word) {   // byte columns 4 word .. 4 word + 3
                u64 part = 0;
#pragma unroll
                for (int b = 3; b >= 0; --b) {
                    u32 d = 0;
#pragma unroll
                    for (int q = 0; q < R::groups; ++q) d = __builtin_amdgcn_udot4(yq[r][q], kResidue<T>.weight[4 * word + b][q], d, false);
                    part = (part << 8) + d;
                }
                sum += (T)part << (32 * word);
            }
            if (row + r < a.M && col + 16 * j < a.N) Zp[(size_t)(row + r) * a.N + col + 16 * j] = sum;
        }
    }
}

// ------------------------------------------------------------------ host ---
// One product is computed block by block so that its fragment stores and residues fit the caller's workspace: `group`
// parties at a time (all, or one), panelsM x panelsN panels of the output at a time, the inner dimension in chunks of
// at most kc.
struct ResiduePlan {
    int group, panelsM, panelsN, totalM, totalN, cols, kc, KT;           // cols: N
    bool narrow;                     // output tiles of 256 x 128 instead of 256 x 256
    bool share;                      // the items beyond the last whole round of workgroups are shared (needs room for parts)
    size_t a_mod, b_mod, a_slot, b_slot, y_bytes;
};

// Products of a few rounds spend much of their time in the last, partly filled one: 2 parties 1000 x 1000 x 5700 (2.25 rounds)
// took 713 us with whole items, 620 with the rest of the items shared; 2 parties 2048^3 over Z_2^128 in the workspace it needs,
// block by block, 2051 and 1795 us.  The parts are reduced modulo p one by one and added when they are combined.
// How many workgroups share an item beyond the last whole round of `grid`: as many as the grid holds, runs of at least
// sixteen k-steps.
inline int parts_of(unsigned items, unsigned grid, int KT)
{
    const unsigned rest = items % grid;
    return rest == 0 ? 1 : (int)std::max(1u, std::min(grid / rest, (unsigned)KT / 8));
}
inline unsigned resident_workgroups(int cus) { return (unsigned)std::max(8, cus / 8 * 8); }
inline size_t tile_bytes_of(bool narrow) { return narrow ? ResidueShape<4>::tile_bytes : ResidueShape<8>::tile_bytes; }

// The most a caller is told to bring for a plan of few blocks (1.8 % of the card's memory), and what it is told to bring for a small
// gain too: 5 parties 4096^3 take 10.95 ms in 3.5 GB and 11.15 in 5.1 GB, 3 parties 4096 x 4096 x 2048 3.53 in 0.9 and 3.52 in 2.1.
constexpr size_t kAmpleWorkspace = (size_t)5 << 30, kModestWorkspace = (size_t)1 << 30;

template <class T> inline size_t plan_bytes(const ResiduePlan &p)
{
    return (size_t)(1 + p.group) * (p.a_slot + p.b_slot) + p.y_bytes;
}
// Output tiles across panels c .. c + pn - 1 (narrow ones only where there are columns).
inline int tiles_across(const ResiduePlan &p, int c, int pn)
{
    return p.narrow ? ceil_div(std::min(p.cols - c * kPanel, pn * kPanel), ResidueShape<4>::BN) : pn;
}
template <class T> inline unsigned plan_items(const ResiduePlan &p)
{
    return (unsigned)(p.group * ResidueTables<T>::L * p.panelsM * tiles_across(p, 0, p.panelsN));
}
template <class T> inline void plan_sizes(ResiduePlan &p, int cus)
{
    constexpr int L = ResidueTables<T>::L;
    p.a_mod = (size_t)p.panelsM * p.KT * kPanelStep;
    p.b_mod = (size_t)p.panelsN * p.KT * kPanelStep;
    p.a_slot = p.a_mod * L;
    p.b_slot = p.b_mod * L;
    p.y_bytes = (size_t)p.group * L * p.panelsM * p.panelsN * kPanel * kPanel;
    const unsigned items = plan_items<T>(p), grid = resident_workgroups(cus);
    if (p.share) p.y_bytes += (size_t)(items % grid) * (parts_of(items, grid, p.KT) - 1) * tile_bytes_of(p.narrow);
}

// Estimated time in microseconds of a plan: k-steps of a tile (256 MFMAs of 16 cycles on four SIMDs), a fixed part per item, the
// bytes of pack and combine as streams, and the three launches with their ramps.  A wave of the pack converts the parties' shares
// one after another, so that a short call over Z_2^128 waits 5 us a party for it (63 us in all at 3 parties 320 x 128 x 96).  Both
// sets are fits to about 2000 products (1 to 8 parties, sides 32 to 8192, wide and narrow tiles, plans of one and of several
// blocks): rms error 5 % over Z_2^64, 8 % over Z_2^128 where the digit kernels are near.
template <class T> struct ResidueCost;
template <> struct ResidueCost<u64> {
    static constexpr double step = 0.661, item = 0.34, narrow_step = 0.608;                          // of a wide tile's
    static constexpr double pack_bytes_per_us = 4.46e6, combine_bytes_per_us = 4.8e6;
    static constexpr double first_block = 11.4, first_block_party = 2.0, block = 13.3, block_party = 2.0;
    static constexpr double shared = 0, shared_part = 2.0;                                           // the combine fetches part by part
};
template <> struct ResidueCost<u128> {
    static constexpr double step = 0.636, item = 0, narrow_step = 0.613;
    static constexpr double pack_bytes_per_us = 4.2e6, combine_bytes_per_us = 4.39e6;
    static constexpr double first_block = 25.2, first_block_party = 4.97, block = 18.2, block_party = 5.43;
    static constexpr double shared = 4.2, shared_part = 7.1;
};
// Taken where its estimate is this much below the digit kernels'.  Against always taking the fastest way the choice, that among the digit kernels
// included, costs 0.5 % over 930 products over Z_2^64 of 3.5e9 ring MACs to 6e10 (2.4 % with the digit kernels estimated as full tiles) and 1.1 %
// over 740 from 4e8 on; and 0.2 % over 8700 over Z_2^128 (1 to 8 parties, sides 16 to 6500), the direct kernel included.
constexpr double kResidueMargin = 0.95;
template <class T> inline double plan_cost(const ResiduePlan &p, int n, int batch, int M, int N, int K, int cus)
{
    using C = ResidueCost<T>;
    constexpr int L = ResidueTables<T>::L;
    const int blocksM = ceil_div(p.totalM, p.panelsM), blocksN = ceil_div(p.totalN, p.panelsN), chunks = ceil_div(K, p.kc);
    const int groups = ceil_div(n, p.group);
    const unsigned items = plan_items<T>(p), grid = resident_workgroups(cus), rest = items % grid;
    const int parts = p.share ? parts_of(items, grid, p.KT) : 1;
    const double step = p.narrow ? C::step * C::narrow_step : C::step, item = p.narrow ? 0 : C::item;
    const double y_bytes = (double)items * tile_bytes_of(p.narrow), part_bytes = (double)rest * (parts - 1) * tile_bytes_of(p.narrow);
    double block_us = items / grid * (2 * p.KT * step + item) + 2 * (y_bytes + part_bytes) / C::combine_bytes_per_us;
    if (rest > 0) block_us += 2 * p.KT * step / parts + item;
    if (parts > 1) block_us += C::shared + C::shared_part * (parts - 1);
    const double blocks = (double)chunks * blocksM * blocksN * groups;
    const bool left_kept = p.group == n;                 // the left triples stay converted across the blocks of a row
    const double w = sizeof(T), padM = (double)p.totalM * kPanel, padN = (double)p.totalN * kPanel;
    const int left_reps = left_kept ? 1 : blocksN, right_reps = left_kept && blocksN == 1 ? 1 : blocksM;
    const double left = (double)K * (M * w * n * (1 + left_reps) + padM * L * (1 + (double)n * left_reps));
    const double right = (double)right_reps * K * (N * w * 2 * n + padN * L * (n + 1));
    const double out = (double)n * M * N * 2 * w * chunks;
    return batch * (blocks * block_us + (left + right) / C::pack_bytes_per_us + out / C::combine_bytes_per_us) + C::first_block +
           C::first_block_party * n + (C::block + C::block_party * p.group) * (blocks * batch - 1);
}

// The cheapest plan that fits `bytes`; false when none does.  For every number of row blocks only the smallest number
// of column blocks that fits is of interest: more blocks only convert more often.
template <class T> inline bool best_plan(int n, int batch, int M, int N, int K, size_t bytes, ResiduePlan &best, double &best_cost)
{
    ResiduePlan p;
    p.totalM = ceil_div(M, kPanel);
    p.totalN = ceil_div(N, kPanel);
    p.cols = N;
    const int chunks = ceil_div(K, ResidueRing<T>::max_k), cus = compute_units();
    p.kc = ceil_div(ceil_div(K, chunks), kStepK) * kStepK;
    p.KT = p.kc / kStepK;
    bool found = false;
    for (int group = n; group >= 1; group = group > 1 ? 1 : 0)
        for (int kind = 0; kind < 4; ++kind) {           // narrow or wide tiles, with or without room for shared items
            p.group = group;
            p.narrow = kind % 2 != 0;
            p.share = kind < 2;
            for (int bm = 1; bm <= std::min(p.totalM, 16); ++bm)
                for (int bn = 1; bn <= std::min(p.totalN, 16); ++bn) {
                    p.panelsM = ceil_div(p.totalM, bm);
                    p.panelsN = ceil_div(p.totalN, bn);
                    plan_sizes<T>(p, cus);
                    if (plan_bytes<T>(p) > bytes) continue;
                    const double c = plan_cost<T>(p, n, batch, M, N, K, cus);
                    if (!found || c < best_cost) { best = p; best_cost = c; found = true; }
                    if (bn == 1) bm = 16;                // whole rows of panels fit: no need for more row blocks
                    break;
                }
        }
    return found;
}

template <class T, int NJ>
spin_status launch_residue_gemm(const ResidueGemmArgs &g, hipStream_t s, const char *where)
{
    static OncePerDevice lds_allowed;
    auto kernel = residue_gemm_kernel<T, NJ>;
    spin_status st = allow_dynamic_lds((const void *)kernel, ResidueShape<NJ>::lds_bytes, lds_allowed);
    if (st != SPIN_OK) return st;
    KernelTimer timer(SPIN_KERNEL_GEMM_RESIDUE, s);
    const unsigned resident = resident_workgroups(compute_units()), most = resident * (kMaxRounds - 1);
    for (unsigned i = 0; i < g.items; i += most) {       // only the last launch has items beyond its whole rounds
        ResidueGemmArgs part = g;
        part.first_item = i;
        part.items = std::min(g.items - i, most);
        part.whole = part.items / resident * resident;
        const unsigned grid = part.whole > 0 ? resident : part.items * (unsigned)part.parts;
        kernel<<<grid, 256, ResidueShape<NJ>::lds_bytes, s>>>(part);
        st = check_launch(where);
        if (st != SPIN_OK) return st;
    }
    return SPIN_OK;
}

template <class T> spin_status run_residue(const MatmulArgsT<T> &a, const ResiduePlan &p, hipStream_t s, const char *where)
{
    constexpr int L = ResidueTables<T>::L;
    char *E = (char *)a.workspace, *A = E + p.a_slot, *F = A + p.group * p.a_slot, *B = F + p.b_slot, *y = B + p.group * p.b_slot;
    const size_t xmat = (size_t)a.M * a.K, ymat = (size_t)a.K * a.N, zmat = (size_t)a.M * a.N;
    const bool vec = a.K % (16 / (int)sizeof(T)) == 0;   // rows 16-byte aligned
    for (int b = 0; b < a.batch; ++b)
        for (int k0 = 0; k0 < a.K; k0 += p.kc)
            for (int r = 0; r < p.totalM; r += p.panelsM)
                for (int c = 0; c < p.totalN; c += p.panelsN)
                    for (int p0 = 0; p0 < a.n; p0 += p.group) {
                        const int k1 = std::min(a.K, k0 + p.kc), KT = ceil_div(k1 - k0, kStepK);
                        const int pm = std::min(p.panelsM, p.totalM - r), pn = std::min(p.panelsN, p.totalN - c);
                        const int last = std::min(a.n, p0 + p.group);
                        const bool all = p.group == a.n, one_c = p.panelsN >= p.totalN;
                        ResiduePackArgs<T> pk;
                        pk.n = a.n;
                        pk.left = ResidueSide<T>{a.X + b * xmat, a.A + b * xmat, a.batch * xmat, a.M, a.K, r * kPanel, k0, k1, E, A,
                                                 p0, last, c == 0 && p0 == 0, pm, KT};
                        pk.right = ResidueSide<T>{a.Y + b * ymat, a.B + b * ymat, a.batch * ymat, a.y_transposed ? a.N : a.K,
                                                  a.y_transposed ? a.K : a.N, c * kPanel, k0, k1, F, B, p0, last, p0 == 0, pn, KT};
                        // with all parties in one group the left operands stay converted across the blocks of a row
                        // of blocks, and the right ones across rows when a row is one block
                        const bool do_left = !(all && c > 0), do_right = !(all && one_c && r > 0);
                        pk.left_blocks = do_left ? residue_pack_blocks<T>(pm, KT) : 0;
                        const unsigned blocks = pk.left_blocks + (do_right ? residue_pack_blocks<T>(pn, KT) : 0);
                        if (blocks > 0) {
                            KernelTimer timer(SPIN_KERNEL_PACK, s);
                            constexpr int threads = 64 * kPackWaves<T>;
                            if constexpr (sizeof(T) == 8) {
                                if (a.y_transposed) {
                                    if (vec) residue_pack_kernel<T, true, true><<<blocks, threads, 0, s>>>(pk);
                                    else residue_pack_kernel<T, false, true><<<blocks, threads, 0, s>>>(pk);
                                } else {
                                    if (vec) residue_pack_kernel<T, true, false><<<blocks, threads, 0, s>>>(pk);
                                    else residue_pack_kernel<T, false, false><<<blocks, threads, 0, s>>>(pk);
                                }
                            } else {
                                residue_pack_kernel<T, true, false><<<blocks, threads, 0, s>>>(pk);
                            }
                            const spin_status st = check_launch(where);
                            if (st != SPIN_OK) return st;
                        }
                        ResidueGemmArgs g{E, A, F, B, (size_t)L * pm * KT * kPanelStep, (size_t)L * pn * KT * kPanelStep,
                                          (size_t)pm * KT * kPanelStep, (size_t)pn * KT * kPanelStep, y, last - p0, L, pm,
                                          tiles_across(p, c, pn), KT, 0, 0, 0, 1, nullptr};
                        const unsigned tiles = (unsigned)(g.tilesM * g.tilesN), resident = resident_workgroups(compute_units());
                        g.items = tiles * L * (unsigned)g.parties;
                        g.y_parts = y + (size_t)g.items * tile_bytes_of(p.narrow);
                        // as many parts as the workspace has room for (blocks at the edge differ from the plan's)
                        const unsigned rest = g.items % resident;
                        const size_t room = ((size_t)((char *)a.workspace + a.workspace_bytes - g.y_parts)) / tile_bytes_of(p.narrow);
                        if (rest > 0 && p.share) g.parts = std::min(parts_of(g.items, resident, KT), 1 + (int)std::min(room / rest, (size_t)1 << 20));
                        spin_status st = p.narrow ? launch_residue_gemm<T, 4>(g, s, where) : launch_residue_gemm<T, 8>(g, s, where);
                        if (st != SPIN_OK) return st;
                        ResidueCombineArgs<T> cb{y, (k0 == 0 ? a.C : a.Z) + ((size_t)p0 * a.batch + b) * zmat,
                                                 a.Z + ((size_t)p0 * a.batch + b) * zmat, a.batch * zmat, a.M, a.N, r * kPanel,
                                                 c * kPanel, g.tilesM, g.tilesN, g.parties, 0, g.y_parts, g.items / resident * resident, g.parts};
                        cb.waves = (unsigned)g.parties * tiles * 4 * (p.narrow ? ResidueShape<4>::stores : ResidueShape<8>::stores);
                        KernelTimer timer(SPIN_KERNEL_COMBINE, s);
                        auto combine = [&](auto nj_c) {
                            constexpr int NJ = decltype(nj_c)::value;
                            if (cb.parts > 1) residue_combine_kernel<T, NJ, true><<<cb.waves / 4, 256, 0, s>>>(cb);
                            else residue_combine_kernel<T, NJ, false><<<cb.waves / 4, 256, 0, s>>>(cb);
                        };
                        if (p.narrow) combine(std::integral_constant<int, 4>());
                        else combine(std::integral_constant<int, 8>());
                        st = check_launch(where);
                        if (st != SPIN_OK) return st;
                    }
    return SPIN_OK;
}

}  // namespace

template <class T>
spin_status launch_matmul_residue(const MatmulArgsT<T> &a, double digit_cost_us, hipStream_t s, const char *where, bool &taken)
{
    ResiduePlan p;
    double cost = 0;
    taken = best_plan<T>(a.n, a.batch, a.M, a.N, a.K, a.workspace_bytes, p, cost) && cost < kResidueMargin * digit_cost_us;
    return taken ? run_residue<T>(a, p, s, where) : SPIN_OK;
}
template spin_status launch_matmul_residue<u64>(const MatmulArgsT<u64> &, double, hipStream_t, const char *, bool &);
template spin_status launch_matmul_residue<u128>(const MatmulArgsT<u128> &, double, hipStream_t, const char *, bool &);

template <class T> size_t residue_workspace_bytes(int n, int batch, int M, int N, int K, size_t need, double digit_cost_us)
{
    ResiduePlan p;
    double cost = 0, most = kResidueMargin * digit_cost_us;
    if (!best_plan<T>(n, batch, M, N, K, kAmpleWorkspace, p, cost) || cost >= most) return 0;
    // beyond what is modest, the smallest plan above the need that is estimated within 1 % of the best
    size_t bytes = plan_bytes<T>(p);
    most = std::min(most, 1.01 * cost);
    while (bytes > kModestWorkspace && best_plan<T>(n, batch, M, N, K, bytes - 1, p, cost) && cost < most && plan_bytes<T>(p) > need)
        bytes = plan_bytes<T>(p);
    return bytes;
}
template size_t residue_workspace_bytes<u64>(int, int, int, int, int, size_t, double);
template size_t residue_workspace_bytes<u128>(int, int, int, int, int, size_t, double);

}  // namespace spin
