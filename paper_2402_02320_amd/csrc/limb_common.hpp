// What the limb-decomposed GEMMs over Z_2^32, Z_2^64 and Z_2^128 share: the balanced-digit conversion, the
// fragment layout and the packs that open E (F) and lay all left (right) operands out as
// int8 MFMA fragments, the direct-to-LDS load, and the mapping of workgroup ids to output tiles.
//
// A ring element of ND bytes (ND = 4, 8 or 16) is rewritten as ND balanced digits s_i in [-128,127] with
// sum_i s_i 256^i == a (mod 2^(8 ND)):  t = a + 0x80..80;  s = t ^ 0x80..80 (bytes read as int8).
// Fragment store: [slot][batch][blk][kt][digit][1024 B]; in one 1 KiB fragment lane l's 16 bytes at
// offset 16 l are digit d of elements (row or column 32 blk + l % 32, k = 32 kt + 16 (l / 32) + 0..15),
// which is exactly one operand of v_mfma_i32_32x32x32_i8.  Zero padded to whole tiles.
#pragma once
#include "common.hpp"

namespace spin {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kFrag = 1024;          // bytes of one 32x32 int8 fragment

__device__ inline void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <class T> __device__ inline T digit_bias();
template <> __device__ inline u32 digit_bias<u32>() { return 0x80808080u; }
template <> __device__ inline u64 digit_bias<u64>() { return 0x8080808080808080ull; }
template <> __device__ inline u128 digit_bias<u128>()
{
    return ((u128)0x8080808080808080ull << 64) | 0x8080808080808080ull;
}
template <class T> __device__ inline T to_digits(T a) { return (a + digit_bias<T>()) ^ digit_bias<T>(); }

// Keeps the compiler from computing v later than here.  Sums over the parties are used last: left alone they are sunk behind the
// stores, and the shares of all parties stay in registers until then (64 registers a party).
template <class T> __device__ inline void computed_here(T &v)
{
    if constexpr (std::is_same<T, u128>::value) {
        u64 low = (u64)v, high = (u64)(v >> 64);
        asm volatile("" : "+v"(low), "+v"(high));
        v = (T)high << 64 | low;
    } else {
        asm volatile("" : "+v"(v));
    }
}

// Transposes 16 digit-words (16 elements x ND digits) into ND rows of 16 bytes and stores row p
// (digit p of the 16 elements) at dst + p*kFrag; NT: with non-temporal stores.
template <class T, bool NT = false> __device__ inline void store_digit_rows(const T (&w)[16], char *dst)
{
#pragma unroll
    for (int word = 0; word < (int)sizeof(T) / 4; ++word) {     // digits 4 word .. 4 word + 3
        u32 rows[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32 w0 = (u32)(w[4 * q + 0] >> (32 * word)), w1 = (u32)(w[4 * q + 1] >> (32 * word));
            u32 w2 = (u32)(w[4 * q + 2] >> (32 * word)), w3 = (u32)(w[4 * q + 3] >> (32 * word));
            // 4x4 byte transpose with v_perm_b32 (selector 0-3: second operand, 4-7: first operand)
            u32 t0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u);   // w0.b0 w1.b0 w0.b1 w1.b1
            u32 t1 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);   // w0.b2 w1.b2 w0.b3 w1.b3
            u32 t2 = __builtin_amdgcn_perm(w3, w2, 0x05010400u);
            u32 t3 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
            rows[0][q] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
            rows[1][q] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
            rows[2][q] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
            rows[3][q] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            v4i v = {(int)rows[p][0], (int)rows[p][1], (int)rows[p][2], (int)rows[p][3]};
            if constexpr (NT) __builtin_nontemporal_store(v, (v4i *)(dst + (size_t)(word * 4 + p) * kFrag));
            else *(v4i *)(dst + (size_t)(word * 4 + p) * kFrag) = v;
        }
    }
}

// Operand sets far larger than the caches are read once and their fragments written once: the pack kernels
// then use non-temporal loads and stores (NT), measured 7 % faster at 5 parties x 4096^2 per side; smaller
// calls keep ordinary accesses so that the GEMM finds the fragments in L2.
constexpr size_t kPackStreamingBytes = (size_t)64 << 20;
template <bool NT, class T> __device__ inline T load_share(const T *p)
{
    if constexpr (NT && sizeof(T) == 8) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT> __device__ inline u64x2 load_share_pair(const u64 *p)
{
    if constexpr (NT) return __builtin_nontemporal_load((const u64x2 *)p);
    else return *(const u64x2 *)p;
}

template <class T> struct PackArgs {
    const T *val;       // X or Y shares   [n][batch][rows][cols]
    const T *tri;       // A or B shares   [n][batch][rows][cols]
    char *pack;         // [n+1][batch][nblk][KT][ND][1024]
    int n, batch;
    int rows, cols;     // source matrix is rows x cols, row-major
    int nblk, KT;       // blocks of 32 along the non-contracted axis; k-tiles of 32
};

// Both pack kernels make one pass over the 2n share streams of their side: the opened matrix (E or F)
// accumulates in registers while each triple share is converted and stored as it arrives.  Slots:
// 0 = opened, 1 + i = party i's triple share (left side A_i; right side B_i, and for party 0 B_0 + F,
// which folds the public E.F term into party 0's first product).  blockIdx.z = batch.  Party 0's triple share is needed again at the end (B_0 + F): rings of
// up to 8 bytes keep it in registers, 16-byte rings read it a second time (KEEP = false) to stay within
// the register file.

// Right side: source K x N row-major, a fragment row is a matrix column, so the 16 consecutive k a
// lane needs are 16 strided loads whose lanes run along contiguous columns.  One wave handles 64
// columns x 16 k (half a k-tile of two adjacent column blocks): every wave-wide load is one contiguous
// 64-element row segment, every store two contiguous half-fragment chunks; consecutive waves continue
// along the row.
// `block` is the workgroup's index within its batch entry b.
// A small pack is bound by what one wave has to issue (one or two waves on a SIMD, 5 cycles an instruction), so the addresses are
// kept off the vector unit: the wave's place is a scalar, every load a scalar row address plus the lane's 32-bit offset, and a
// tile inside the matrix is not masked.  With all parties' loads behind one another and 64-bit vector addresses and divisions a
// wave of three parties took 14.5 us (rows) and 8 us (columns), now 5.3 and 6; whole calls of 420 small products over the three
// rings: 2.4 to 4.7 % less time, up to 25 % where eight parties' shares had spilled.
template <int NP, class T, int WAVES, bool NT>
__device__ __forceinline__ void pack_right_body(const PackArgs<T> &a, unsigned block, int b)
{
    constexpr int ND = sizeof(T);
    constexpr bool KEEP = sizeof(T) <= 8;
    const int lane = threadIdx.x % 64;
    const unsigned nblk2 = (unsigned)(a.nblk + 1) / 2;     // pairs of column blocks
    const unsigned tile = block * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);   // (kt, half, block pair), block pair fastest
    const unsigned kt2 = tile / nblk2;
    if (kt2 >= 2u * (unsigned)a.KT) return;
    const int blk2 = (int)(tile - kt2 * nblk2), half = (int)(kt2 % 2), kt = (int)(kt2 / 2);
    const int blk = blk2 * 2 + lane / 32;
    const int K = a.rows, N = a.cols;
    const int col0 = min(blk2 * 64, N - 1), k0 = kt * 32 + 16 * half, row0 = min(k0, K - 1);
    const bool owns = blk < a.nblk;                        // the last pair may have only one block
    const bool inside = blk2 * 64 + 64 <= N && k0 + 16 <= K;                     // uniform
    const bool col_ok = blk2 * 64 + lane < N;
    const size_t mat = (size_t)K * N;
    const size_t party_stride = (size_t)a.batch * mat;
    const size_t base = (size_t)b * mat + (size_t)row0 * N + col0;
    const u32 lane_off = (u32)(min(blk2 * 64 + lane, N - 1) - col0);
    auto frag = [&](int slot) -> char * {
        return a.pack + ((((size_t)slot * a.batch + b) * a.nblk + blk) * a.KT + kt) * (ND * kFrag) +
               (lane % 32 + 32 * half) * 16;
    };
    // Loads are unconditional (an element outside the matrix reads one inside and is replaced by zero when it is stored):
    // guarded by a branch each, every load would be awaited before the next one is issued.
    auto load = [&](const T *matrix, T (&v)[16]) {
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = load_share<NT>(matrix + (base + (size_t)(min(k0 + j, K - 1) - row0) * N) + lane_off);
    };
    auto store = [&](T (&v)[16], int slot) {
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = to_digits<T>(v[j]);
        if (!inside) {
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = col_ok && k0 + j < K ? v[j] : (T)0;
        }
        if (owns) store_digit_rows<T, NT>(v, frag(slot));
    };
    T opened[16], first[KEEP ? 16 : 1], tv[2][16], xv[2][16];
#pragma unroll
    for (int j = 0; j < 16; ++j) opened[j] = 0;
    load(a.tri, tv[0]);
    load(a.val, xv[0]);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        constexpr int kAhead = KEEP ? 1 : 0;
        const int cur = i % 2 * kAhead, nxt = (i + 1) % 2 * kAhead;
        if (KEEP && i + 1 < NP) {
            load(a.tri + (i + 1) * party_stride, tv[nxt]);
            load(a.val + (i + 1) * party_stride, xv[nxt]);
        }
        if (KEEP) __builtin_amdgcn_sched_barrier(0);       // one party's loads in flight, not all of them: they would not fit the registers
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            opened[j] += xv[cur][j] - tv[cur][j];
            if (NP > 1) computed_here(opened[j]);
        }
        if (i == 0) {
            if constexpr (KEEP) {
#pragma unroll
                for (int j = 0; j < 16; ++j) first[j] = tv[cur][j];
            }
        } else {
            store(tv[cur], i + 1);
        }
        if (!KEEP && i + 1 < NP) {
            load(a.tri + (i + 1) * party_stride, tv[nxt]);
            load(a.val + (i + 1) * party_stride, xv[nxt]);
        }
    }
    T w[16];
    if constexpr (KEEP) {
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = first[j] + opened[j];
    } else {
        load(a.tri, w);
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] += opened[j];
    }
    store(opened, 0);
    store(w, 1);
}
template <int WAVES> __host__ __device__ inline unsigned pack_right_blocks(int nblk, int KT)
{
    return (unsigned)(((long)((nblk + 1) / 2) * KT * 2 + WAVES - 1) / WAVES);
}

// Several products of different shapes in one launch (the grouped call): the descriptors travel as a kernel
// argument, every workgroup looks its group up from the table of first workgroup ids.
constexpr int kGroupsPerLaunch = 32;
template <class Args> struct GroupTable {
    int count;
    unsigned first[kGroupsPerLaunch + 1];                  // first workgroup id of every group, then the total
    Args e[kGroupsPerLaunch];
};
template <class Args> __device__ inline int group_of(const GroupTable<Args> &t, unsigned id)
{
    int g = 0;
    for (int i = 1; i < t.count; ++i) g += id >= t.first[i] ? 1 : 0;
    return g;
}

// Left side: source M x K row-major, a fragment row is a matrix row.  Reading 16 consecutive k per
// lane directly would make every wave-wide load touch 64 different rows; instead a wave reads its
// 32 x 32 tile (blk, kt) as whole-row segments (16 bytes per lane, 32 k of one row contiguous), sums the parties'
// shares in that layout, and turns each 32 x 32 tile through LDS (rows padded by 16 bytes,
// conflict-free for 16-byte accesses both ways) so that each lane ends up with the 16 consecutive k
// of one row that a fragment chunk needs.  WAVES = waves per block (LDS: WAVES x 32 padded rows).
// `right` packs a right operand that is stored transposed ([N][K] row-major, the layout of K in
// Q.K^T): the access pattern is the left side's, the slot rule the right side's (party 0's slot holds
// B_0 + F).
template <class T> constexpr int turn_row_bytes = 32 * sizeof(T) + 16;       // one row of the LDS turn

template <int NP, class T, bool VEC, int WAVES, bool NT>
__device__ __forceinline__ void pack_left_body(const PackArgs<T> &a, unsigned block, int b, char *lds, bool right)
{
    constexpr int ND = sizeof(T);
    constexpr bool KEEP = sizeof(T) <= 8;
    constexpr int EPL = 16 / ND;                 // elements per 16-byte lane load: 4, 2 or 1
    constexpr int LPR = 32 / EPL;                // lanes that cover the 32 k of one row: 8, 16 or 32
    constexpr int RPL = 64 / LPR;                // rows per wave-wide load: 8, 4 or 2
    constexpr int NL = 32 / RPL;                 // loads per lane: 4, 8 or 16
    constexpr int kRowBytes = turn_row_bytes<T>;
    struct alignas(16) Pair { T e[EPL]; };
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const unsigned tile = block * WAVES + wave;             // (blk, kt) pair
    const int blk = (int)(tile / (unsigned)a.KT), kt = (int)(tile - (unsigned)blk * (unsigned)a.KT);
    if (blk >= a.nblk) return;                              // whole waves leave; each works in its own part of LDS
    const int M = a.rows, K = a.cols;
    const size_t mat = (size_t)M * K;
    const size_t party_stride = (size_t)a.batch * mat;
    const int kk = kt * 32 + EPL * (lane % LPR);            // this lane's k (pair) of every row it loads
    const int row0 = blk * 32 + lane / LPR;                 // and the first of them
    const bool inside = blk * 32 + 32 <= M && kt * 32 + 32 <= K;                 // uniform
    // Elements outside the matrix read one inside, so that no load sits behind a branch and has to be awaited before the next is
    // issued; they become zero before they are stored.  Offsets are 64 bits: 32 rows may be longer than 4 GiB.  One and two parties
    // over 16-byte rings compute them anew for every matrix, from a number of columns that the compiler cannot tell to be the same:
    // kept, they take 32 registers, and two parties spill four at two waves a SIMD.  (More parties have one wave and room for them;
    // computed anew they cost eight parties 8 x 64^3 2 % of the call.)
    constexpr bool OFFSETS_ANEW = sizeof(T) == 16 && NP <= 2;
    auto offset = [&](int j, int cols) -> size_t { return (size_t)min(row0 + RPL * j, M - 1) * cols + min(kk, VEC ? K - EPL : K - 1); };
    size_t off[OFFSETS_ANEW ? 1 : NL];
#pragma unroll
    for (int j = 0; j < (OFFSETS_ANEW ? 0 : NL); ++j) off[j] = offset(j, K);
    auto load = [&](const T *matrices, int i, Pair (&v)[NL]) {
        const T *base = matrices + ((size_t)i * party_stride + (size_t)b * mat);
        int cols = K;
        if (OFFSETS_ANEW) asm volatile("" : "+s"(cols));
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const size_t at = OFFSETS_ANEW ? offset(j, cols) : off[j];
            if constexpr (VEC) {
                if constexpr (NT && sizeof(T) == 8) {
                    const u64x2 two = load_share_pair<true>((const u64 *)(base + at));
                    v[j].e[0] = two.x;
                    v[j].e[1] = two.y;
                } else {
                    v[j] = *(const Pair *)(base + at);
                }
            } else {
#pragma unroll
                for (int q = 0; q < EPL; ++q) v[j].e[q] = load_share<NT>(base + at + (kk + q < K ? q : 0));
            }
        }
    };
    // lane -> LDS: written as (row RPL j + lane / LPR, k position lane % LPR), read back as
    // (row lane % 32, k 16 (lane / 32) ..)
    char *mine = lds + wave * (32 * kRowBytes);
    auto turn_and_store = [&](const Pair (&v)[NL], int slot) {
        wait_lds();                                         // the previous round's reads are done (one wave, in order)
        Pair d[NL];
#pragma unroll
        for (int j = 0; j < NL; ++j)
#pragma unroll
            for (int q = 0; q < EPL; ++q) d[j].e[q] = to_digits<T>(v[j].e[q]);
        if (!inside) {
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int q = 0; q < EPL; ++q) d[j].e[q] = row0 + RPL * j < M && kk + q < K ? d[j].e[q] : (T)0;
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) *(Pair *)(mine + (RPL * j + lane / LPR) * kRowBytes + (lane % LPR) * 16) = d[j];
        wait_lds();
        T w[16];
#pragma unroll
        for (int j = 0; j < 16 / EPL; ++j) {
            Pair p = *(const Pair *)(mine + (lane % 32) * kRowBytes + (lane / 32) * (16 * ND) + j * 16);
#pragma unroll
            for (int q = 0; q < EPL; ++q) w[EPL * j + q] = p.e[q];
        }
        store_digit_rows<T, NT>(w, a.pack + ((((size_t)slot * a.batch + b) * a.nblk + blk) * a.KT + kt) * (ND * kFrag) + lane * 16);
    };

    Pair opened[NL], first[KEEP ? NL : 1];
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
        for (int q = 0; q < EPL; ++q) opened[j].e[q] = 0;
    // The next party's loads are in flight while one is turned; all of them at once would not fit the registers.  16-byte rings have no
    // room for that, and keep the loop rolled.
    constexpr int kPartyUnroll = KEEP ? NP : 1;
    Pair tv[KEEP ? 2 : 1][NL], xv[KEEP ? 2 : 1][NL];
    if constexpr (KEEP) {
        load(a.tri, 0, tv[0]);
        load(a.val, 0, xv[0]);
    }
#pragma unroll kPartyUnroll
    for (int i = 0; i < NP; ++i) {
        const int cur = KEEP ? i % 2 : 0;
        if constexpr (KEEP) {
            if (i + 1 < NP) {
                load(a.tri, i + 1, tv[cur ^ 1]);
                load(a.val, i + 1, xv[cur ^ 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
            load(a.tri, i, tv[0]);
            load(a.val, i, xv[0]);
        }
#pragma unroll
        for (int j = 0; j < NL; ++j)
#pragma unroll
            for (int q = 0; q < EPL; ++q) {
                opened[j].e[q] += xv[cur][j].e[q] - tv[cur][j].e[q];
                if (NP > 1) computed_here(opened[j].e[q]);
            }
        if (i == 0) {
            if constexpr (KEEP) {
#pragma unroll
                for (int j = 0; j < NL; ++j) first[j] = tv[cur][j];
            }
        } else {
            turn_and_store(tv[cur], i + 1);
        }
    }
    turn_and_store(opened, 0);
    if constexpr (KEEP) {
        if (right) {
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int q = 0; q < EPL; ++q) first[j].e[q] += opened[j].e[q];
        }
        turn_and_store(first, 1);
    } else {
        load(a.tri, 0, tv[0]);
        if (right) {
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int q = 0; q < EPL; ++q) tv[0][j].e[q] += opened[j].e[q];
        }
        turn_and_store(tv[0], 1);
    }
}
template <int WAVES> __host__ __device__ inline unsigned pack_left_blocks(int nblk, int KT) { return (unsigned)(((long)nblk * KT + WAVES - 1) / WAVES); }

// The packs of one product: left operands, right ones, and the copy Z = C where several workgroups will add onto a tile
// of Z.  Small ones go out as one launch (kBoth): workgroups 0 .. left_blocks - 1 of a batch entry pack left operands, the
// next right_blocks right ones, the last copy_blocks copy.  The parts are independent and each of them alone leaves most of
// the chip idle at the sizes where a launch counts: a layer of 4 parties, 250 x 301 x 785, where they were three launches of
// 12.8 + 9.8 + 3.3 us, went from 60.5 to 49.6 us, one of 2 parties, 1024^3, from 162.7 to 158.5 us.
// Streaming ones (kPackStreamingBytes) have a launch a part, with non-temporal accesses.
enum PackSide { kBoth, kLeft, kRight };
template <class T> struct PackLaunch {
    PackArgs<T> left, right;
    const T *copy_from;
    T *copy_to;
    size_t copy_count;                                   // elements, all parties and batch entries
    unsigned left_blocks, right_blocks, copy_blocks;     // per batch entry
};
template <class T> constexpr int pack_waves = sizeof(T) <= 8 ? 4 : 2;
constexpr int kCopyPerThread = 8;
// Two waves on a SIMD wherever that costs no spilled registers (24 to 48 of them, 3 to 7 % of a call, at the others).  No kernel here
// may spill: where a spilled group of four registers lies partly in spare registers and partly in memory, the compiler (clang 22 of
// ROCm 7.2) can lose one of the parts.  Eight parties' left pack with the shares of all parties in flight spilled 56; the
// reload of rows 24 .. 27 of party 0's shares set one register of two, and E was wrong in those rows.
template <int NP, class T> constexpr int pack_waves_per_simd = (sizeof(T) == 16 ? NP > 2 : NP > 6) ? 1 : 2;

template <int NP, class T, bool VEC, bool TRANSPOSED, bool NT, PackSide SIDE>
__global__ __launch_bounds__(64 * pack_waves<T>, (pack_waves_per_simd<NP, T>)) void pack_kernel(PackLaunch<T> a)
{
    constexpr int WAVES = pack_waves<T>;
    __shared__ __attribute__((aligned(16))) char lds[SIDE == kRight && !TRANSPOSED ? 16 : WAVES * 32 * turn_row_bytes<T>];
    unsigned block = blockIdx.x;
    if (SIDE == kLeft || (SIDE == kBoth && block < a.left_blocks)) {
        pack_left_body<NP, T, VEC, WAVES, NT>(a.left, block, blockIdx.z, lds, false);
    } else if (SIDE == kRight || (block -= a.left_blocks) < a.right_blocks) {
        if constexpr (TRANSPOSED) pack_left_body<NP, T, VEC, WAVES, NT>(a.right, block, blockIdx.z, lds, true);
        else pack_right_body<NP, T, WAVES, NT>(a.right, block, blockIdx.z);
    } else {
        block -= a.right_blocks;
        size_t i = ((size_t)blockIdx.z * a.copy_blocks + block) * (64 * WAVES * kCopyPerThread) + threadIdx.x;
#pragma unroll
        for (int u = 0; u < kCopyPerThread; ++u, i += 64 * WAVES)
            if (i < a.copy_count) a.copy_to[i] = a.copy_from[i];
    }
}

// The same for several products of different shapes: every entry of the table is one side of one product.  Six attention
// products of 3 parties, with three pack launches of 10.3 + 10.3 + 9.4 us before: 69.1 -> 52.4 us a
// call (39.7 with their GEMMs in one launch too).
struct GroupedPackSide {
    PackArgs<u64> a;
    int kind;                                            // 0, 1: left (16-byte rows or not); 2, 3: transposed right; 4: right
};
template <int NP>
__global__ __launch_bounds__(256, (pack_waves_per_simd<NP, u64>)) void pack_grouped_kernel(GroupTable<GroupedPackSide> t)
{
    __shared__ __attribute__((aligned(16))) char lds[4 * 32 * turn_row_bytes<u64>];
    const int gi = group_of(t, blockIdx.x);
    const PackArgs<u64> a = t.e[gi].a;
    const int kind = t.e[gi].kind;
    const unsigned local = blockIdx.x - t.first[gi];
    const unsigned per_batch = kind == 4 ? pack_right_blocks<4>(a.nblk, a.KT) : pack_left_blocks<4>(a.nblk, a.KT);
    const unsigned block = local % per_batch;
    const int b = (int)(local / per_batch);
    if (kind == 0 || kind == 2) pack_left_body<NP, u64, true, 4, false>(a, block, b, lds, kind == 2);
    else if (kind == 1 || kind == 3) pack_left_body<NP, u64, false, 4, false>(a, block, b, lds, kind == 3);
    else pack_right_body<NP, u64, 4, false>(a, block, b);
}

// One direct-to-LDS load: 64 lanes x 16 bytes from src + lane*16 to the LDS address lds_dst + lane*16.
// Issued through inline assembly so that the compiler's LDS-DMA bookkeeping does not serialise the
// software pipeline; completion is awaited explicitly (wait_loads) before the workgroup barrier.
// The instruction takes its LDS base from m0, a register the compiler reserves for its own use and
// does not accept in a clobber list, so the statement puts back the value it found there (m0 is read
// when the load issues, so restoring it right after is safe).
__device__ inline void load_fragment_to_lds(const char *src, u32 lds_dst, u32 lane16)
{
    u32 saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "v"(lane16), "s"(src), "s"(lds_dst) : "memory");
}
template <int N> __device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
__device__ inline void workgroup_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Output tile of a workgroup.  Workgroup ids are dealt round-robin to the 8 XCDs; each XCD gets a
// contiguous range of the work items, so that workgroups sharing an L2 also share operand fragments,
// and walks the tiles of a matrix in 4-tile-tall column strips.
__device__ inline long xcd_contiguous_id(long id, long total)
{
    const long chunk = (total + 7) / 8;
    const long full = total - (chunk - 1) * 8;       // XCDs that own `chunk` items (the rest own chunk-1)
    const int xcd = (int)(id % 8);
    const long within = id / 8;
    return xcd < full ? xcd * chunk + within : full * chunk + (xcd - full) * (chunk - 1) + within;
}
struct TileId { int pb, tm, tn; };     // party * batch + b, tile row, tile column
__device__ inline TileId tile_of(long id, int tilesM, int tilesN)
{
    const int per_mat = tilesM * tilesN;
    TileId r;
    r.pb = (int)(id / per_mat);
    int t = (int)(id % per_mat);
    constexpr int GROUP = 4;
    const int strip = t / (GROUP * tilesN);
    const int strip_h = min(GROUP, tilesM - strip * GROUP);
    t -= strip * GROUP * tilesN;
    r.tm = strip * GROUP + t % strip_h;
    r.tn = t / strip_h;
    return r;
}
__device__ inline TileId map_tile(long id, int tilesM, int tilesN, long total)
{
    return tile_of(xcd_contiguous_id(id, total), tilesM, tilesN);
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Operand sets beyond the caches (kPackStreamingBytes per side) use non-temporal accesses.
template <class T> inline bool pack_streams(int n, int batch, int rows, int cols)
{
    return (size_t)n * batch * rows * cols * sizeof(T) >= kPackStreamingBytes;
}

template <class T, PackSide SIDE> inline void launch_pack_part(const MatmulArgsT<T> &a, const PackLaunch<T> &p, bool nt, hipStream_t s)
{
    constexpr int threads = 64 * pack_waves<T>;
    const bool vec = a.K % (16 / (int)sizeof(T)) == 0;   // rows 16-byte aligned
    const unsigned blocks = SIDE == kLeft ? p.left_blocks : SIDE == kRight ? p.right_blocks : p.left_blocks + p.right_blocks + p.copy_blocks;
    const dim3 grid(blocks, 1, a.batch);
    for_party_count(a.n, [&](auto np) {
        constexpr int NP = decltype(np)::value;
        auto go = [&](auto vec_c, auto transposed_c) {
            constexpr bool VEC = decltype(vec_c)::value, TRANSPOSED = decltype(transposed_c)::value;
            if constexpr (SIDE != kBoth) {               // products that stream past the caches have a launch a side
                if (nt) {
                    pack_kernel<NP, T, VEC, TRANSPOSED, true, SIDE><<<grid, threads, 0, s>>>(p);
                    return;
                }
            }
            pack_kernel<NP, T, VEC, TRANSPOSED, false, SIDE><<<grid, threads, 0, s>>>(p);
        };
        if constexpr (sizeof(T) == 8 && SIDE != kLeft) { // only the 64-bit calls take a transposed right operand
            if (a.y_transposed) {
                if (vec) go(std::true_type(), std::true_type());
                else go(std::false_type(), std::true_type());
                return;
            }
        }
        if constexpr (sizeof(T) == 16 || SIDE == kRight) {                   // alignment of rows is all the same
            go(std::true_type(), std::false_type());
        } else {
            if (vec) go(std::true_type(), std::false_type());
            else go(std::false_type(), std::false_type());
        }
    });
}

// The copy rides along up to this size of C: at the occupancy of the packs it is slower than a launch of its own (5 parties 1024^3,
// 42 MB: 388 us a call with it in the pack, 364 without; 3 parties over Z_2^32, 16384 x 128 x 576, 25 MB: 169 and 164; 8 parties 700 x
// 500 x 300, 22 MB: 115 and 122).
constexpr size_t kCopyWithPackBytes = (size_t)23 << 20;
// Where only one of the sides streams, the copy goes with the other, which is then short: 7 parties over Z_2^32, 2880 x 128 x 1440, 10
// MB: 177 us a call with it, 170 without; 5 parties 2000 x 100 x 1000, 8 MB: 147 and 150.
constexpr size_t kCopyWithSideBytes = (size_t)8 << 20;

// Packs the left operands (X, A; unless packA is null) and the right ones (Y, B) of one Beaver matmul.  Where copy_c is set and
// one of its launches can take the copy of C to Z along, that is done too; returns whether it was.
template <class T>
inline bool launch_pack(const MatmulArgsT<T> &a, char *packA, char *packB, int nblkA, int nblkB, int KT, bool copy_c, hipStream_t s)
{
    KernelTimer timer(SPIN_KERNEL_PACK, s);
    constexpr int WAVES = pack_waves<T>;
    PackLaunch<T> p{};
    p.left = PackArgs<T>{a.X, a.A, packA, a.n, a.batch, a.M, a.K, nblkA, KT};
    if (a.y_transposed) p.right = PackArgs<T>{a.Y, a.B, packB, a.n, a.batch, a.N, a.K, nblkB, KT};
    else p.right = PackArgs<T>{a.Y, a.B, packB, a.n, a.batch, a.K, a.N, nblkB, KT};
    p.left_blocks = packA ? pack_left_blocks<WAVES>(nblkA, KT) : 0;
    p.right_blocks = a.y_transposed ? pack_left_blocks<WAVES>(nblkB, KT) : pack_right_blocks<WAVES>(nblkB, KT);
    const bool nt_left = pack_streams<T>(a.n, a.batch, a.M, a.K), nt_right = pack_streams<T>(a.n, a.batch, a.K, a.N);
    const bool both = p.left_blocks > 0 && !nt_left && !nt_right;
    const size_t count = (size_t)a.n * a.batch * a.M * a.N, per_block = 64 * WAVES * kCopyPerThread;
    copy_c = copy_c && count * sizeof(T) <= (both ? kCopyWithPackBytes : kCopyWithSideBytes) && !(nt_left && nt_right);
    if (copy_c) {
        p.copy_from = a.C;
        p.copy_to = a.Z;
        p.copy_count = count;
        p.copy_blocks = (unsigned)(((count + per_block - 1) / per_block + a.batch - 1) / a.batch);
    }
    if (both) {
        launch_pack_part<T, kBoth>(a, p, false, s);
        return copy_c;
    }
    // the copy goes with a side that does not stream, in the kernel of both with no workgroups for the other side
    const bool copy_left = copy_c && !nt_left && p.left_blocks > 0, copy_right = copy_c && !copy_left;
    PackLaunch<T> one = p;
    if (copy_left) {
        one.right_blocks = 0;
        launch_pack_part<T, kBoth>(a, one, false, s);
    } else if (p.left_blocks > 0) {
        launch_pack_part<T, kLeft>(a, p, nt_left, s);
    }
    if (copy_right) {
        p.left_blocks = 0;
        launch_pack_part<T, kBoth>(a, p, false, s);
    } else {
        launch_pack_part<T, kRight>(a, p, nt_right, s);
    }
    return copy_c;
}

}  // namespace
}  // namespace spin
