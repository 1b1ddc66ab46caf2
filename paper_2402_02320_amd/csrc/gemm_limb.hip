// Exact ring GEMM over Z_2^64 (and, with four digits, Z_2^32) on the int8 matrix cores.
//
// Z_2^64: every uint64 a is rewritten as eight balanced digits s_0..s_7 in [-128,127]
// with  sum_i s_i 256^i == a  (mod 2^64)   [t = a + 0x80..80; s = t ^ 0x80..80].
// Then  a*b == sum_{i+j<=7} s_i t_j 256^(i+j)  (mod 2^64): the 28 digit pairs
// with i+j >= 8 are multiples of 2^64.  The 36 surviving pairs are int8 x int8
// products; pairs of one diagonal d = i+j share an int32 MFMA accumulator D_d,
// and the result is  sum_d (int64)D_d << 8d  (mod 2^64).
//
// int32 headroom: |s_i t_j| <= 2^14.  D_d needs 64-8d exact bits, so only
// d <= 3 must not overflow: (d+1) * Ktot * 2^14 < 2^31  <=>  Ktot < 2^15.
// For d >= 4 only the low 32 bits matter and the accumulators wrap (two's
// complement), which leaves those bits right.  The host splits the inner
// dimension into chunks of at most 511 k-tiles per operand pair.
//
// Z_2^32 (the Fixed32 representation of Section 7.1): four digits, the 10 pairs with i+j <= 3, four
// diagonals; every diagonal needs at most 32 exact bits, so wrapping accumulators are always right
// and the inner dimension is never split.
//
// Kernels:
//  pack_kernel (limb_common.hpp)  opens E and F, converts E, A_i and F, B_i' to digits and stores them as 1 KiB MFMA
//                fragments: both sides in one launch.
//  limb_gemm_kernel  per party: Z_i = C_i + [E | A_i] . [B_i' ; F], fragments
//                streamed global -> LDS with direct-to-LDS loads, 36 MFMAs per
//                32x32x32 step into 8 diagonal accumulators, recombined once.
//  limb_gemm_rows_kernel  products with few column tiles (N <= 64; attention shapes), at most three
//                parties: no left pack at all -- the workgroup opens E from the raw X_j, A_j itself, converts E and the A_p to
//                fragments in LDS and multiplies all parties' outputs of a row block.
//  *_grouped_kernel  the same bodies for several products of different shapes in one launch
//                (spin_beaver_matmul_grouped), the products found through a table in the kernel arguments.
// Larger products go to the residue GEMM (gemm_residue.hip; over Z_2^32 to gemm_strassen.hip) and the smallest to one launch of vector arithmetic
// (gemm_direct.hip); digit_route's estimate is this file's side of those choices.
#include <algorithm>
#include <cmath>
#include <vector>

#include "limb_common.hpp"

namespace spin {
namespace {

// Per ring: the largest workgroup tile (waves are 2 x 2, each WM x WN MFMA tiles of 32 x 32; ND * WM * WN * 16 accumulator
// registers <= 256) and the longest run of k-tiles one launch may accumulate.
template <class T> struct Ring;
template <> struct Ring<u64> {
    static constexpr int WM = 2, WN = 1;
    static constexpr int max_chunk_tiles = 511;        // 2*511*32 = 32704 < 2^15 digit products per accumulator
};
template <> struct Ring<u32> {
    static constexpr int WM = 2, WN = 2;
    static constexpr int max_chunk_tiles = 1 << 20;    // no headroom limit; keeps the step count an int
};
// Of a wave with UNITS = WM * WN MFMA tiles of ND digits: the interleave of one k-step (slots = MFMA index within the step), an LDS read after
// every rd_every-th MFMA from slot 0 and a direct-to-LDS load after every ld_every-th from slot ld_first; the LDS stages; and the waves on a
// SIMD, one of each workgroup that a CU then holds.
template <int ND, int UNITS> struct Interleave;
template <> struct Interleave<8, 2> { static constexpr int rd_every = 2, ld_first = 13, ld_every = 4, stages = 3, waves = 1; };   // 72 MFMAs, 24 reads, 12 loads
template <> struct Interleave<8, 1> { static constexpr int rd_every = 1, ld_first = 17, ld_every = 2, stages = 2, waves = 2; };   // 36, 16, 8
template <> struct Interleave<4, 4> { static constexpr int rd_every = 2, ld_first = 5, ld_every = 4, stages = 3, waves = 1; };    // 40, 16, 8
template <> struct Interleave<4, 2> { static constexpr int rd_every = 1, ld_first = 8, ld_every = 2, stages = 3, waves = 2; };    // 20, 12, 6
template <> struct Interleave<4, 1> { static constexpr int rd_every = 1, ld_first = 1, ld_every = 2, stages = 3, waves = 3; };    // 10, 8, 4

// ------------------------------------------------------------------ GEMM ---
template <class T> struct GemmArgs {
    const char *packA;   // [n+1][batch][nblkA][KT][ND][1024]: slot 0 = E, slot 1+i = A_i
    const char *packB;   // [n+1][batch][nblkB][KT][ND][1024]: slot 0 = F, slot 1+i = B_i'
    const T *C;          // [n][batch][M][N]  (or Z itself for the later k-chunks); null: nothing to add
    T *Z;
    int n, batch, M, N;
    int nblkA, nblkB, KT;
    int kt0, ktn;        // this launch covers k-tiles [kt0, kt0+ktn) of both operand pairs
    int tilesM, tilesN;
    int splits;          // workgroups per output tile: each takes split_steps of the 2*ktn k-steps and, when
    int split_steps;     // splits > 1, adds its part onto Z atomically (Z then starts out as C)
};

template <class T, int WM_ = Ring<T>::WM, int WN_ = Ring<T>::WN>
struct GemmShape {
    static constexpr int ND = sizeof(T);                         // digits per ring element
    static constexpr int WM = WM_, WN = WN_;
    using Slots = Interleave<ND, WM * WN>;
    static constexpr int NSTAGE = Slots::stages;                 // LDS ring: one stage read, the others in flight
    static constexpr int BM = 2 * 32 * WM, BN = 2 * 32 * WN;     // 4 waves as 2 x 2
    static constexpr int FA = BM / 32 * ND, FB = BN / 32 * ND;
    static constexpr int stage_bytes = (FA + FB) * kFrag;
    static constexpr int lds_bytes = NSTAGE * stage_bytes;
    static constexpr int loads_per_wave = (FA + FB) / 4;
    static constexpr int frags_per_wave = (WM + WN) * ND;        // LDS -> register reads per step
    static constexpr int mfma_per_step = ND * (ND + 1) / 2 * WM * WN;
    static_assert(ND * WM * WN * 16 <= 256, "accumulators exceed the AGPR file");
};

// sum_d D_d 256^d (mod 2^(8 ND)) of the diagonal sums D_d held as int32: the low four diagonals as signed
// 64-bit multiply-adds (256^d fits an int32), the high four only reach the upper word, where they are plain
// 32-bit shifts and adds.  About ten instructions per element where shifting every sign-extended term
// through 64 bits takes forty.
__device__ inline u64 recombine_diagonals(int d0, int d1, int d2, int d3, int d4, int d5, int d6, int d7)
{
    long long low = (long long)d0;
    low += (long long)d1 * (1 << 8);
    low += (long long)d2 * (1 << 16);
    low += (long long)d3 * (1 << 24);
    const u32 high = (u32)((u64)low >> 32) + (u32)d4 + ((u32)d5 << 8) + ((u32)d6 << 16) + ((u32)d7 << 24);
    return ((u64)high << 32) | (u32)low;
}
__device__ inline u32 recombine_diagonals(int d0, int d1, int d2, int d3)
{
    return (u32)d0 + ((u32)d1 << 8) + ((u32)d2 << 16) + ((u32)d3 << 24);
}

__device__ inline void ring_atomic_add(u64 *p, u64 v) { atomicAdd((unsigned long long *)p, (unsigned long long)v); }
__device__ inline void ring_atomic_add(u32 *p, u32 v) { atomicAdd((unsigned int *)p, (unsigned int)v); }

// Pipeline (per wave; step s covers one 32-deep k-tile of one operand pair; counts for Z_2^64):
//   G(s)  12 direct-to-LDS loads of this wave's share of step s into LDS stage s % 3
//   R(s)  24 ds_read_b128 of the wave's fragments of step s into registers
//   M(s)  72 MFMAs of step s
// Iteration s: [wait G(s+1); barrier]  then M(s) interleaved with R(s+1) and G(s+3).
// The barrier at the top of iteration s also tells every wave that all R(s) are done, so stage s % 3
// can be refilled by G(s+3).  Two groups of loads are in flight while a step computes.
template <class T, class S = GemmShape<T>>
__device__ __forceinline__ void limb_gemm_body(const GemmArgs<T> &g, unsigned block)
{
    constexpr int kDigits = S::ND, WM = S::WM, WN = S::WN;
    extern __shared__ __attribute__((aligned(1024))) char lds[];

    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wm = wave / 2, wn = wave % 2;

    // work item = (split, tile), tiles fastest: neighbours on an XCD work on neighbouring tiles of one k-range
    const long tiles_total = (long)g.tilesM * g.tilesN * g.n * g.batch;
    const long item = xcd_contiguous_id(block, tiles_total * g.splits);
    const int split = (int)(item / tiles_total);
    const TileId tile = tile_of(item % tiles_total, g.tilesM, g.tilesN);
    const int pb = tile.pb, tm = tile.tm, tn = tile.tn;
    const int party = pb / g.batch, b = pb % g.batch;

    // fragment streams: step < ktn uses (E, B_i'), step >= ktn uses (A_i, F)
    const size_t slotA = (size_t)g.batch * g.nblkA * g.KT * (kDigits * kFrag);
    const size_t slotB = (size_t)g.batch * g.nblkB * g.KT * (kDigits * kFrag);
    const char *a_first = g.packA + (size_t)b * g.nblkA * g.KT * (kDigits * kFrag);   // E
    const char *a_second = a_first + (size_t)(1 + party) * slotA;                      // A_i
    const char *b_second = g.packB + (size_t)b * g.nblkB * g.KT * (kDigits * kFrag);  // F
    const char *b_first = b_second + (size_t)(1 + party) * slotB;                      // B_i'

    // this workgroup's k-steps [s0, s0 + steps) of the 2 * ktn (both counts even)
    const int s0 = split * g.split_steps;
    const int steps = min(g.split_steps, 2 * g.ktn - s0);
    const bool starts_in_second = s0 >= g.ktn;
    const u32 lds0 = (u32)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const u32 lane16 = lane * 16;

    // Load cursor: where the loads of the next step to be fetched come from and go to.  It lives on
    // the scalar unit and advances by one k-tile per step (no division, no per-load selects); at the
    // switch from the first operand pair to the second it jumps to the other fragment streams.
    // This wave loads fragments f = 4q + wave, q < loads_per_wave: row/column block f / ND = q / (ND/4)
    // of the tile and digit f % ND = 4 (q % (ND/4)) + wave, so only q-dependent constants remain per load.
    const size_t blk_stride = (size_t)g.KT * (kDigits * kFrag);
    const size_t kt0_off = (size_t)g.kt0 * (kDigits * kFrag) + wave * kFrag;
    const char *second_a = a_second + (size_t)tm * (S::BM / 32) * blk_stride + kt0_off;
    const char *second_b = b_second + (size_t)tn * (S::BN / 32) * blk_stride + kt0_off;
    const size_t start_off = (size_t)(starts_in_second ? s0 - g.ktn : s0) * (kDigits * kFrag);
    const char *ld_a = (starts_in_second ? second_a : a_first + (size_t)tm * (S::BM / 32) * blk_stride + kt0_off) + start_off;
    const char *ld_b = (starts_in_second ? second_b : b_first + (size_t)tn * (S::BN / 32) * blk_stride + kt0_off) + start_off;
    int ld_left = starts_in_second ? 0x7fffffff : g.ktn - s0;   // steps until the cursor switches operand pair
    u32 ld_lds = lds0 + wave * kFrag;                    // LDS destination of the cursor's stage
    const u32 lds_wrap = lds0 + wave * kFrag + (S::NSTAGE - 1) * S::stage_bytes;
    auto issue_load = [&](int q) {                       // q is a compile-time constant after unrolling
        constexpr int qa = S::FA / 4;                    // loads of left-operand fragments per wave
        constexpr int per_blk = kDigits / 4;             // loads of this wave per 32-row (32-column) block
        const char *p = q < qa ? ld_a + (size_t)(q / per_blk) * blk_stride + (q % per_blk) * (4 * kFrag)
                               : ld_b + (size_t)((q - qa) / per_blk) * blk_stride + ((q - qa) % per_blk) * (4 * kFrag);
        load_fragment_to_lds(p, ld_lds + q * (4 * kFrag), lane16);
    };
    auto advance_load_cursor = [&]() {
        ld_a += kDigits * kFrag;
        ld_b += kDigits * kFrag;
        if (--ld_left == 0) { ld_a = second_a; ld_b = second_b; }
        ld_lds = ld_lds == lds_wrap ? lds_wrap - (S::NSTAGE - 1) * S::stage_bytes : ld_lds + S::stage_bytes;
    };

    v16i acc[WM][WN][kDigits];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int d = 0; d < kDigits; ++d) acc[i][j][d] = (v16i)(0);

    // fragment registers, double buffered: [buffer][B fragments then A fragments]; the read cursor
    // (two LDS pointers of this wave within the stage to be read next) cycles through the stages
    v4i fr[2][S::frags_per_wave];
    const char *rd_a = lds + (wm * WM * kDigits) * kFrag + lane16;
    const char *rd_b = lds + (S::FA + wn * WN * kDigits) * kFrag + lane16;
    const char *rd_wrap = rd_a + (S::NSTAGE - 1) * S::stage_bytes;
    auto read_fragment = [&](int q) -> v4i {             // q < WN*8: B fragment q; else A fragment q - WN*8
        return *(const v4i *)(q < WN * kDigits ? rd_b + q * kFrag : rd_a + (q - WN * kDigits) * kFrag);
    };
    auto advance_read_cursor = [&]() {
        const bool wrap = rd_a == rd_wrap;
        rd_a = wrap ? rd_a - (S::NSTAGE - 1) * S::stage_bytes : rd_a + S::stage_bytes;
        rd_b = wrap ? rd_b - (S::NSTAGE - 1) * S::stage_bytes : rd_b + S::stage_bytes;
    };

    // prologue: G(0), G(1), G(2); R(0)
#pragma unroll
    for (int q = 0; q < S::loads_per_wave; ++q) issue_load(q);
    advance_load_cursor();
#pragma unroll
    for (int q = 0; q < S::loads_per_wave; ++q) issue_load(q);
    advance_load_cursor();
    if (S::NSTAGE == 3 && steps > 2) {
#pragma unroll
        for (int q = 0; q < S::loads_per_wave; ++q) issue_load(q);
        advance_load_cursor();
        wait_loads<2 * S::loads_per_wave>();
    } else {
        wait_loads<S::loads_per_wave>();
    }
    workgroup_barrier();
#pragma unroll
    for (int q = 0; q < S::frags_per_wave; ++q) fr[0][q] = read_fragment(q);
    advance_read_cursor();

    // One step.  CUR: register buffer holding this step.  LOAD: the step that fills this step's stage exists (three or, of two stages,
    // two ahead).  NEXT: the next step exists.  MORE: the step two ahead exists (of three stages its loads stay in flight across the wait).
    auto iteration = [&](auto cur_c, auto load_c, auto next_c, auto more_c) {
        constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
        constexpr bool LOAD = decltype(load_c)::value, NEXT = decltype(next_c)::value, MORE = decltype(more_c)::value;
        if (NEXT) {
            if (MORE) wait_loads<(S::NSTAGE - 2) * S::loads_per_wave>(); else wait_loads<0>();
        }
        wait_lds();
        workgroup_barrier();
        int slot = 0;
#pragma unroll
        for (int da = 0; da < kDigits; ++da)
#pragma unroll
            for (int db = 0; db + da < kDigits; ++db)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        acc[i][j][da + db] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
                            fr[cur][WN * kDigits + i * kDigits + da], fr[cur][j * kDigits + db], acc[i][j][da + db],
                            0, 0, 0);
                        // Between the MFMAs: the next step's LDS reads (every rd_every-th slot from the
                        // start, so they are done long before the next barrier), the global loads of the
                        // step three ahead (every ld_every-th slot from ld_first), and the two cursor
                        // updates, so that the last MFMAs of a step and the barrier that follows have no
                        // scalar work between them.  sched_barrier pins this order: left alone, the
                        // scheduler sinks each read next to its first use and the MFMA pipe then waits
                        // out the LDS latency.
                        constexpr int rd_every = S::Slots::rd_every;
                        constexpr int rd_last = rd_every * (S::frags_per_wave - 1);
                        constexpr int ld_first = S::Slots::ld_first;
                        constexpr int ld_every = S::Slots::ld_every;
                        constexpr int ld_last = ld_first + ld_every * (S::loads_per_wave - 1);
                        static_assert(rd_every >= 1 && ld_every >= 1 && ld_last + 1 < S::mfma_per_step &&
                                      rd_last + 1 < S::mfma_per_step, "tile too small for this interleave");
                        if (NEXT && slot % rd_every == 0 && slot <= rd_last) {
                            fr[nxt][slot / rd_every] = read_fragment(slot / rd_every);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (NEXT && slot == rd_last + 1) {
                            advance_read_cursor();
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (LOAD && slot >= ld_first && (slot - ld_first) % ld_every == 0 && slot <= ld_last) {
                            issue_load((slot - ld_first) / ld_every);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (LOAD && slot == ld_last + 1) {
                            advance_load_cursor();
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        ++slot;
                    }
    };
    using Y = std::true_type;
    using F = std::false_type;
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    int s = 0;
    for (; s + 4 < steps; s += 2) {                       // steps is even; both halves have all neighbours
        iteration(B0(), Y(), Y(), Y());
        iteration(B1(), Y(), Y(), Y());
    }
    using LastLoad = std::integral_constant<bool, S::NSTAGE == 2>;
    if (steps >= 4) {
        iteration(B0(), Y(), Y(), Y());                   // step steps-4: loads the last step (of two stages: the one before)
        iteration(B1(), LastLoad(), Y(), Y());
    }
    iteration(B0(), F(), Y(), F());                       // step steps-2

    // C_i is fetched under the last step (the fragment buffer that step would have filled is free), so that
    // the epilogue starts with its operands at hand instead of a memory round trip with nothing else on the
    // CU.  Rows and columns beyond the matrix are redirected to its last row / column; what they bring is
    // never stored.  C and Z may be the same buffer: every element is read and written by the same lane.
    // With several workgroups per tile (splits > 1) Z already holds C and every part is added atomically:
    // ring addition is associative and commutative, so the result does not depend on the order of arrival.
    const size_t mat = (size_t)g.M * g.N;
    const T *Cm = g.C + (size_t)pb * mat;
    T *Zm = g.Z + (size_t)pb * mat;
    const bool interior = (tm + 1) * S::BM <= g.M && (tn + 1) * S::BN <= g.N;     // uniform over the workgroup
    const bool atomic = g.splits > 1, no_c = atomic || g.C == nullptr;
    T cv[WM][WN][16];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            const int col = min(tn * S::BN + (wn * WN + j) * 32 + lane % 32, g.N - 1);
            const int row0 = tm * S::BM + (wm * WM + i) * 32 + 4 * (lane / 32);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                cv[i][j][r] = no_c ? (T)0 : Cm[(size_t)min(row0 + 8 * (r / 4) + r % 4, g.M - 1) * g.N + col];
        }
    __builtin_amdgcn_sched_barrier(0);
    iteration(B1(), F(), F(), F());                       // step steps-1

    // Recombine the diagonals and add C_i.
    // Tiles that lie wholly inside the matrix take branch-free stores: with a bounds check per element every
    // store sits in a basic block of its own and waits for the one before.
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {                   // one 32 x 32 MFMA tile at a time
            const int col = tn * S::BN + (wn * WN + j) * 32 + lane % 32;
            const int row0 = tm * S::BM + (wm * WM + i) * 32 + 4 * (lane / 32);
            auto row_of = [&](int r) { return row0 + 8 * (r / 4) + r % 4; };
            T v[16];
            __builtin_amdgcn_sched_barrier(0);           // keeps the scheduler from hoisting the next tile's work
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = cv[i][j][r];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if constexpr (kDigits == 8)
                    v[r] += recombine_diagonals(acc[i][j][0][r], acc[i][j][1][r], acc[i][j][2][r], acc[i][j][3][r],
                                                acc[i][j][4 % kDigits][r], acc[i][j][5 % kDigits][r],
                                                acc[i][j][6 % kDigits][r], acc[i][j][7 % kDigits][r]);
                else
                    v[r] += recombine_diagonals(acc[i][j][0][r], acc[i][j][1][r], acc[i][j][2][r], acc[i][j][3][r]);
            }
            if (atomic) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (interior || (row_of(r) < g.M && col < g.N)) ring_atomic_add(Zm + (size_t)row_of(r) * g.N + col, v[r]);
            } else if (interior) {
#pragma unroll
                for (int r = 0; r < 16; ++r) Zm[(size_t)row_of(r) * g.N + col] = v[r];
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (row_of(r) < g.M && col < g.N) Zm[(size_t)row_of(r) * g.N + col] = v[r];
            }
        }
}

template <class T, class S = GemmShape<T>>
__global__ __launch_bounds__(256, (S::Slots::waves)) void limb_gemm_kernel(GemmArgs<T> g)
{
    limb_gemm_body<T, S>(g, blockIdx.x);
}

// Products of different shapes in one launch (the grouped call): every workgroup finds its product in the table.
template <class T, class S>
__global__ __launch_bounds__(256, (S::Slots::waves)) void limb_gemm_grouped_kernel(GroupTable<GemmArgs<T>> t)
{
    const int gi = group_of(t, blockIdx.x);
    limb_gemm_body<T, S>(t.e[gi], blockIdx.x - t.first[gi]);
}

// ------------------------------------------------- row-streaming GEMM ---
// Z_2^64 products whose output is a single column tile (N <= 64): every left fragment would be used by
// exactly one output tile, so writing the left operands out as fragments and reading them back (the pack
// pre-pass) costs more HBM traffic than the product itself.  Here the left fragments never exist in
// memory.  (Products of a few column tiles and a short inner dimension -- the attention shapes -- take the
// same kernel once per column tile when that is cheaper than the pre-pass: the raw shares are then read once
// per column tile, from L2.)  One workgroup owns a block of 32 rows and one column tile of 64 for ALL
// parties (NP <= 3) and walks the inner dimension once.
//
// What has to be multiplied per k-tile of 32 is 2 NP units of 32 x 32 outputs (party, column half), twice: E . B_p' and A_p . F,
// 36 MFMAs each.  Eight waves share it, two to a SIMD and 256 registers each, so that one's waits are covered by the other's MFMAs,
// and so that every SIMD has the same number of MFMAs: a unit is one wave's, with all eight diagonal accumulators, or two waves', 18
// MFMAs and four diagonals each (0, 1, 6, 7 and 2, 3, 4, 5; no accumulator exists twice, and the two parts are added through LDS at the end).
//   NP = 3: units 0 .. 3 whole (waves 0 .. 3), units 4 and 5 in parts (waves 4 .. 7): 54 MFMAs a SIMD and half step, where one
//           wave per party on three SIMDs had 72;   NP = 2: four units in parts;   NP = 1: two units in parts (waves 0 .. 3).
// Besides,
//   waves 0 .. 3 ("loaders")     bring the right fragments (packed beforehand: they are small, shared by all row blocks and stay in
//       L2) into two LDS stages with direct-to-LDS loads, three half steps ahead;
//   waves 4 .. 7 ("converters")  load the raw shares of X_j and A_j into registers two k-tiles ahead (each byte of the left operands
//       is read exactly once: 8 rows x 256 bytes per wave), open E = sum_j (X_j - A_j), convert E and every A_p to digits
//       and write them to LDS as fragments.
// A half step is one operand pair of one k-tile and ends with the workgroup's barrier.  In the first half of tile t all waves read
// E(t) and B'(t) and the converters write A(t); in the second they read A(t) and F(t) and the converters open and write
// E(t + 1): so E and A need one stage each, which with two of B' and F is all 160 KB of a CU at three parties.
// Nothing is masked at ragged edges: loads that would leave the matrix are redirected inside it, and what they bring
// only meets zero-padded rows of the right fragments (k >= K) or lands in output rows that are never stored (row >= M).
// A launch has at most one workgroup per CU (more would only queue: a workgroup takes a whole CU); each walks
// its share of the (row block, column tile) items, and t above counts the k-tiles of all its items in one
// sequence (an odd KT padded by a tile without products, so that a tile's parity tells its registers and stage): loads and conversions
// run ahead across item boundaries, under the recombination and the stores of the item before.
//
// Measured against one wave per party, which converted its A_p between its MFMAs and read right fragments from L2 into registers half a step
// ahead, and a producer wave for E (whole calls, the pack included): 3 parties 12262 x 59 x 125 59.0 -> 41.3 us, 20000 x 50 x 125 77.9 ->
// 58.3, 64 entries of 128 x 128 x 64 (keys transposed) 38.1 -> 32.1, of 128 x 64 x 128 34.2 -> 30.8; 2 parties 20 entries of 100^3 25.5 ->
// 20.8, 131072 x 64 x 576 847 -> 792.  3 parties 131072 x 64 x 576 stay at 1120: its 3.6 GB take 770 us with nothing multiplied, its products 700 with
// nothing loaded; together L2 is busy 0.96 of the cycles (9.1 GB asked of it, 4.8 of them right fragments that every row block reads again, at 7.7
// TB/s) and the matrix pipes 0.54, and the clock is down at 1.2 to 1.65 GHz.  With shares one k-tile ahead (40 registers fewer) the first two
// take 44.8 and 62.1 us.
// Workgroups of a row-kernel launch: (row blocks over all batch entries, rounded up to a multiple of 8) x column tiles.
__host__ __device__ inline long rows_grid(int batch, int M, int tilesN)
{
    const long rblocks = (long)batch * ((M + 31) / 32);
    return (rblocks + 7) / 8 * 8 * tilesN;
}

struct RowGemmArgs {
    const u64 *X, *A;        // [n][batch][M][K]
    const char *packB;       // right fragment store [n+1][batch][2 tilesN][KT][8][1024]: slot 0 = F, 1 + i = B_i'
    const u64 *C;            // [n][batch][M][N]
    u64 *Z;
    int batch, M, N, K, KT, tilesN;
};

typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) const v4i lds_v4i;
typedef __attribute__((address_space(3))) u32 lds_u32;
typedef __attribute__((address_space(3))) u64 lds_u64;

constexpr int kRowThreads = 512;
template <int NP> struct RowLds {
    static constexpr int unit = 8 * kFrag;                           // the eight digits of 32 rows (columns) and 32 k
    static constexpr int e = 0, a = unit;                            // E; A_p
    static constexpr int b = a + NP * unit, b_stage = 2 * NP * unit; // B_p', two column blocks each, two stages
    static constexpr int f = b + 2 * b_stage, f_stage = 2 * unit;    // F
    static constexpr int halved = NP == 3 ? 2 : 2 * NP;              // units in two parts: 8 KB of partial sums each,
    static constexpr int sums = NP == 3 ? a : f + 2 * f_stage;       // over A_p where nothing else is left (16 of 24 KB)
    static constexpr int bytes = NP == 3 ? f + 2 * f_stage : sums + halved * unit;
};
static_assert(RowLds<3>::bytes <= 160 * 1024 && RowLds<2>::bytes <= 160 * 1024, "one CU's LDS");

// The balanced digits of four elements, transposed: out[d] = digit d of elements 0 .. 3.
__device__ inline void digit_quads(const u64 (&v)[4], u32 (&out)[8])
{
    u64 s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = to_digits<u64>(v[i]);
#pragma unroll
    for (int word = 0; word < 2; ++word) {
        const u32 w0 = (u32)(s[0] >> (32 * word)), w1 = (u32)(s[1] >> (32 * word));
        const u32 w2 = (u32)(s[2] >> (32 * word)), w3 = (u32)(s[3] >> (32 * word));
        const u32 t0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), t1 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
        const u32 t2 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), t3 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
        out[4 * word + 0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
        out[4 * word + 1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
        out[4 * word + 2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
        out[4 * word + 3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
    }
}

// Part of a unit that a wave multiplies: all diagonals, or those of one of two waves with 18 of the 36 digit pairs each.
enum RowPart { kWholeUnit, kDiagonals0167, kDiagonals2345, kNoUnit };
constexpr bool in_part(RowPart part, int d)
{
    const bool inner = d >= 2 && d <= 5;
    return part == kWholeUnit || (part == kDiagonals2345 && inner) || (part == kDiagonals0167 && !inner);
}

// One wave of the row kernel.  unit = 2 party + column half; VEC: rows of X and A are 16-byte aligned (even K).
template <int NP, bool VEC, bool CONVERTS, RowPart PART>
__device__ __forceinline__ void rows_wave(const RowGemmArgs &g, unsigned first_item, unsigned item_stride, int n_items, unsigned share0,
                                          int wave, int unit, int sums_slot, lds_char *lds)
{
    using L = RowLds<NP>;
    const int lane = threadIdx.x % 64;
    const u32 lane16 = lane * 16;
    const int KT = g.KT, KT2 = (KT + 1) & ~1, total = n_items * KT2;
    const unsigned rblocks = (unsigned)((g.M + 31) / 32);
    const int party = unit / 2, half = unit % 2;
    struct Place { int b, rb, tn; };
    auto place_of = [&](unsigned item) {
        const unsigned q = item / 8, rblock = share0 + q / (unsigned)g.tilesN;
        return Place{(int)(rblock / rblocks), (int)(rblock % rblocks), (int)(q % (unsigned)g.tilesN)};
    };
    const unsigned last_item = first_item + (unsigned)(n_items - 1) * item_stride;

    // ---- loaders: F runs one k-tile ahead of the products, B' two.  (For the tile that pads an odd KT the one before it is loaded again.)
    const size_t cb_stride = (size_t)KT * L::unit;                   // from a column block to the next
    const size_t slot_stride = (size_t)g.batch * g.tilesN * 2 * cb_stride;
    struct Cursor { unsigned item; int kt; const char *at; u32 stage; };
    const u32 lds0 = (u32)(uintptr_t)lds + wave * kFrag;
    auto cursor_base = [&](unsigned item) -> const char * {
        const Place p = place_of(item);
        return g.packB + ((size_t)p.b * g.tilesN + p.tn) * 2 * cb_stride + wave * kFrag;
    };
    auto advance = [&](Cursor &c) {
        c.stage ^= 1;
        ++c.kt;
        if (c.kt < KT) c.at += L::unit;
        if (c.kt == KT2) {
            c.kt = 0;
            c.item += item_stride;                                   // past the last item nothing is loaded
            c.at = cursor_base(c.item);
        }
    };
    auto load_blocks = [&](const char *src, u32 dst) {               // this wave's quarter of two column blocks
#pragma unroll
        for (int q = 0; q < 4; ++q) load_fragment_to_lds(src + (q / 2) * cb_stride + (q % 2) * (4 * kFrag), dst + (q / 2) * L::unit + (q % 2) * (4 * kFrag), lane16);
    };
    auto load_f = [&](Cursor &c) {
        load_blocks(c.at, lds0 + L::f + c.stage * L::f_stage);
        advance(c);
    };
    auto load_b = [&](Cursor &c) {
#pragma unroll
        for (int p = 0; p < NP; ++p) load_blocks(c.at + (size_t)(1 + p) * slot_stride, lds0 + L::b + c.stage * L::b_stage + p * (2 * L::unit));
        advance(c);
    };
    // After the loads that a half step waits for, at most one load_f and one load_b were issued; loads return in order.
    constexpr int kInFlight = 4 + 4 * NP;

    // ---- converters: lane (row 8 (wave % 4) + lane / 8, k 4 (lane % 8) ..) of the 32 x 32 tile
    const int c_row = 8 * (wave % 4) + lane / 8, c_k = 4 * (lane % 8);
    const size_t pitch = (size_t)g.K * 8, party_stride = (size_t)g.batch * g.M * pitch;
    struct Shares { u64 e[NP][4]; } x[2], a[2];                      // of even and of odd tiles
    struct Rows { unsigned item; int kt; size_t tile; u32 off; };
    auto set_rows = [&](Rows &c) {
        const Place p = place_of(min(c.item, last_item));
        c.tile = ((size_t)p.b * g.M + (size_t)p.rb * 32) * pitch;    // of party 0, the row block's first row and k = 0
        c.off = (u32)min(c_row, g.M - 1 - p.rb * 32) * (u32)pitch + c_k * 8;      // K < 2^15: below 2^24
    };
    // Nothing is fetched for the tile that pads an odd KT nor past the last item: the loads are issued all the same, of no bytes, so that
    // the compiler can tell how many are in flight behind the ones that it waits for.
    auto load_shares = [&](const u64 *matrix, Rows &c, Shares &v) {
        const u32 size = c.kt < KT && c.item <= last_item ? 0x7fffffffu : 0u;
        u32 off[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) off[i] = c.kt * 32 + c_k + i < g.K ? c.off + 8 * i : 0;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((char *)matrix + (c.tile + j * party_stride), 0, size, 0x00020000);
            if constexpr (VEC) {
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    const v4i two = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rsrc, off[i], c.kt * 256, 0);
                    v.e[j][i] = (u64)(u32)two.y << 32 | (u32)two.x;
                    v.e[j][i + 1] = (u64)(u32)two.w << 32 | (u32)two.z;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const auto one = __builtin_amdgcn_raw_buffer_load_b64(rsrc, off[i], c.kt * 256, 0);
                    v.e[j][i] = (u64)(u32)one[1] << 32 | (u32)one[0];
                }
            }
        }
        if (++c.kt == KT2) {
            c.kt = 0;
            c.item += item_stride;
            set_rows(c);
        }
    };
    lds_char *quad = lds + (c_row + 32 * (c_k / 16)) * 16 + c_k % 16;
    auto write_digits = [&](const u64 (&v)[4], int at) {
        u32 d[8];
        digit_quads(v, d);
#pragma unroll
        for (int i = 0; i < 8; ++i) *(lds_u32 *)(quad + at + i * kFrag) = d[i];
    };
    auto open_left = [&](const Shares &xs, const Shares &as) {
        u64 e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            e[i] = xs.e[0][i] - as.e[0][i];
#pragma unroll
            for (int j = 1; j < NP; ++j) e[i] += xs.e[j][i] - as.e[j][i];
        }
        write_digits(e, L::e);
    };

    // ---- products
    v16i acc[8];
    auto multiply = [&](int left_at, int right_at) {
        if constexpr (PART != kNoUnit) {
            u32 l16 = lane16;                                        // the addresses made anew: kept, they take six registers
            asm volatile("" : "+v"(l16));
            lds_char *left = lds + left_at + l16, *right = lds + right_at + l16;
            constexpr int digits = PART == kDiagonals2345 ? 6 : 8;
            if constexpr (PART == kWholeUnit) {
                v4i l[digits], r[digits];
#pragma unroll
                for (int m = 0; m < digits; ++m) {
                    r[m] = *(lds_v4i *)(right + m * kFrag);
                    l[m] = *(lds_v4i *)(left + m * kFrag);
                }
                __builtin_amdgcn_sched_barrier(0);
                // in the order in which the fragments arrive: after 2 m of them m^2 pairs are there
#pragma unroll
                for (int m = 0; m < digits; ++m)
#pragma unroll
                    for (int o = 0; o < 2 * m + 1; ++o) {
                        const int da = o <= m ? m : o - m - 1, db = o <= m ? o : m;
                        if (da + db < 8) acc[da + db] = __builtin_amdgcn_mfma_i32_32x32x32_i8(l[da], r[db], acc[da + db], 0, 0, 0);
                    }
            } else {                                                 // the raw shares leave room for the right fragments and two left ones
                v4i r[digits], l[2];
                l[0] = *(lds_v4i *)left;
#pragma unroll
                for (int m = 0; m < digits; ++m) r[m] = *(lds_v4i *)(right + m * kFrag);
#pragma unroll
                for (int da = 0; da < digits; ++da) {
                    if (da + 1 < digits) l[(da + 1) % 2] = *(lds_v4i *)(left + (da + 1) * kFrag);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int db = 0; db < digits; ++db)
                        if (da + db < 8 && in_part(PART, da + db))
                            acc[da + db] = __builtin_amdgcn_mfma_i32_32x32x32_i8(l[da % 2], r[db], acc[da + db], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);                       // products are not moved behind the half step's barrier
        }
    };
    const int e_at = L::e, a_at = L::a + party * L::unit, b_at = L::b + unit * L::unit, f_at = L::f + half * L::unit;

    // ---- start: B'(0), F(0), B'(1); E(0)
    Cursor cf{first_item, 0, nullptr, 0}, cb{first_item, 0, nullptr, 0};
    Rows cx{first_item, 0, 0, 0}, ca{first_item, 0, 0, 0};
    if constexpr (!CONVERTS) {
        cf.at = cb.at = cursor_base(first_item);
        load_b(cb);
        load_f(cf);
        load_b(cb);
        wait_loads<kInFlight>();
    } else {
        set_rows(cx);
        set_rows(ca);
        load_shares(g.X, cx, x[0]);
        load_shares(g.A, ca, a[0]);
        load_shares(g.X, cx, x[1]);
        load_shares(g.A, ca, a[1]);
        open_left(x[0], a[0]);
        load_shares(g.X, cx, x[0]);
    }
    wait_lds();
    workgroup_barrier();

    int t = 0;
    unsigned item_id = first_item;
    for (int item = 0; item < n_items; ++item, item_id += item_stride) {
        const Place p = place_of(item_id);
        const size_t zmat = (size_t)g.M * g.N;
        const size_t block0 = ((size_t)party * g.batch + p.b) * zmat + (size_t)p.rb * 32 * g.N;
        const char *Cm = (const char *)(g.C + block0);               // the item's rows; 32 of them are below 4 GiB (N <= 2^24)
        char *Zm = (char *)(g.Z + block0);
        const bool interior = (p.rb + 1) * 32 <= g.M && (p.tn + 1) * 64 <= g.N;
        const int rows = g.M - p.rb * 32, col0 = p.tn * 64 + half * 32;
        // Where the lane's outputs are, from a number of columns and a lane number that the compiler cannot tell to be the same twice: kept
        // between C and Z, and from item to item, the offsets would take 17 registers that are not there.
        struct Outputs {
            int row0, col;
            u32 cols;
            __device__ int row(int r) const { return row0 + 8 * (r / 4) + r % 4; }
            __device__ u32 at(int row, int column) const { return ((u32)row * cols + (u32)column) * 8u; }
        };
        auto outputs = [&]() {
            int c = g.N, l;
            asm volatile("" : "+s"(c));
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
            return Outputs{4 * (l / 32), col0 + l % 32, (u32)c};
        };
        u64 v[16];
        auto load_c = [&]() {
            const Outputs o = outputs();
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = *(const u64 *)(Cm + o.at(min(o.row(r), rows - 1), min(o.col, g.N - 1)));
        };
#pragma unroll
        for (int d = 0; d < 8; ++d) acc[d] = (v16i)(0);
        // one k-tile; ODD: its parity in the sequence, and so its LDS stage and its registers
        auto tile = [&](auto odd_c, int kt) {
            constexpr int ODD = decltype(odd_c)::value;
            const bool real = !ODD || kt < KT;
            // E . B_p'
            if constexpr (CONVERTS) {
#pragma unroll
                for (int j = 0; j < NP; ++j) write_digits(a[ODD].e[j], L::a + j * L::unit);
                load_shares(g.A, ca, a[ODD]);                        // of tile t + 2
            } else {
                if (t + 1 < total) load_f(cf);
            }
            if (real) multiply(e_at, b_at + ODD * L::b_stage);
            if constexpr (!CONVERTS) {
                if (t + 2 < total) wait_loads<kInFlight>(); else wait_loads<0>();        // F(t)
            }
            wait_lds();
            workgroup_barrier();
            // A_p . F
            if constexpr (CONVERTS) {
                open_left(x[ODD ^ 1], a[ODD ^ 1]);
                load_shares(g.X, cx, x[ODD ^ 1]);                    // of tile t + 3
            } else {
                if (t + 2 < total) load_b(cb);
            }
            // C_p is fetched under the item's last products.  Rows and columns beyond the matrix are redirected to its last row /
            // column; what they bring is never stored.  C may be Z itself: every element is read and written by the same lane.
            if constexpr (ODD && PART == kWholeUnit) {
                if (kt + 1 == KT2) load_c();
            }
            if (real) multiply(a_at, f_at + ODD * L::f_stage);
            if constexpr (!CONVERTS) {
                if (t + 2 < total) wait_loads<kInFlight>(); else wait_loads<0>();        // B'(t + 1)
            }
            wait_lds();
            workgroup_barrier();
            ++t;
        };
        for (int kt = 0; kt < KT2; kt += 2) {
            tile(std::integral_constant<int, 0>(), kt);
            tile(std::integral_constant<int, 1>(), kt + 1);
        }
        // the two parts of a halved unit meet in LDS
        lds_char *sums = lds + L::sums + sums_slot * L::unit + lane * 8;
        u64 w[16];
        if constexpr (PART == kDiagonals2345) {
#pragma unroll
            for (int r = 0; r < 16; ++r) *(lds_u64 *)(sums + r * 512) = recombine_diagonals(0, 0, acc[2][r], acc[3][r], acc[4][r], acc[5][r], 0, 0);
            wait_lds();
        }
        workgroup_barrier();
        if constexpr (PART == kDiagonals0167) {
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = *(lds_u64 *)(sums + r * 512) + recombine_diagonals(acc[0][r], acc[1][r], 0, 0, 0, 0, acc[6][r], acc[7][r]);
            wait_lds();
            __builtin_amdgcn_sched_barrier(0);
            load_c();                                                // into the accumulators' registers: there are no others
        }
        if (NP == 3) workgroup_barrier();                            // the sums lie where A_p goes next
        if constexpr (PART == kWholeUnit || PART == kDiagonals0167) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (PART == kWholeUnit) v[r] += recombine_diagonals(acc[0][r], acc[1][r], acc[2][r], acc[3][r], acc[4][r], acc[5][r], acc[6][r], acc[7][r]);
                else v[r] += w[r];
            }
            const Outputs o = outputs();
            if (interior) {
#pragma unroll
                for (int r = 0; r < 16; ++r) *(u64 *)(Zm + o.at(o.row(r), o.col)) = v[r];
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (o.row(r) < rows && o.col < g.N) *(u64 *)(Zm + o.at(o.row(r), o.col)) = v[r];
            }
        }
    }
}

template <int NP, bool VEC>
__device__ __forceinline__ void limb_gemm_rows_body(const RowGemmArgs &g, unsigned first_item, unsigned item_stride)
{
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    lds_char *lds = (lds_char *)lds_raw;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // Workgroup ids are dealt round-robin to the 8 XCDs, and an XCD gets a contiguous eighth of the row blocks (counted over all batch
    // entries), column tiles fastest: the column tiles of a row block meet in one L2, where the raw shares come from memory once,
    // and so do the row blocks of a batch entry, for its right fragments.  (Row blocks dealt one by one: every entry's right fragments
    // went to up to eight L2s.  64 entries of 3 parties, 128 x 128 x 64: 44.6 us a call instead of 40.2.)
    // A workgroup walks the items first_item, first_item + item_stride, ... (the stride is a multiple of 8, so all
    // of them belong to one XCD); rows_grid pads the id space to 8 equal shares, and a workgroup that has none leaves at once.
    // Item i = column tile (i / 8) % tilesN of row block i / 8 / tilesN of share i % 8 (all counts are below 2^31, which the
    // host checks).
    const unsigned rblocks_all = (unsigned)g.batch * (unsigned)((g.M + 31) / 32);
    const unsigned share = first_item % 8;
    const unsigned share0 = (unsigned)((u64)rblocks_all * share / 8), share1 = (unsigned)((u64)rblocks_all * (share + 1) / 8);
    const unsigned limit = (share1 - share0) * 8 * (unsigned)g.tilesN;
    const int n_items = first_item < limit ? (int)((limit - 1 - first_item) / item_stride) + 1 : 0;
    if (n_items == 0) return;                            // all waves together
    auto go = [&](auto converts, auto part, int unit, int sums_slot) {
        rows_wave<NP, VEC, decltype(converts)::value, decltype(part)::value>(g, first_item, item_stride, n_items, share0, wave, unit, sums_slot, lds);
    };
    using Loads = std::false_type;
    using Converts = std::true_type;
    using Whole = std::integral_constant<RowPart, kWholeUnit>;
    using PartA = std::integral_constant<RowPart, kDiagonals0167>;
    using PartB = std::integral_constant<RowPart, kDiagonals2345>;
    using None = std::integral_constant<RowPart, kNoUnit>;
    if constexpr (NP == 3) {
        const int pair = (wave - 4) / 2;
        if (wave < 4) go(Loads(), Whole(), wave, 0);
        else if (wave % 2 == 0) go(Converts(), PartA(), 4 + pair, pair);
        else go(Converts(), PartB(), 4 + pair, pair);
    } else {
        const int pair = wave / 2;
        if (wave < 4) {
            if (wave % 2 == 0) go(Loads(), PartA(), pair, pair);
            else go(Loads(), PartB(), pair, pair);
        } else if (NP == 1) {
            go(Converts(), None(), 0, 0);
        } else if (wave % 2 == 0) {
            go(Converts(), PartA(), pair, pair);
        } else {
            go(Converts(), PartB(), pair, pair);
        }
    }
}

template <int NP, bool VEC>
__global__ __launch_bounds__(kRowThreads) void limb_gemm_rows_kernel(RowGemmArgs g)
{
    limb_gemm_rows_body<NP, VEC>(g, blockIdx.x, gridDim.x);
}

template <int NP>
__global__ __launch_bounds__(kRowThreads) void limb_gemm_rows_grouped_kernel(GroupTable<RowGemmArgs> t)
{
    const int gi = group_of(t, blockIdx.x);
    if (t.e[gi].K % 2 == 0) limb_gemm_rows_body<NP, true>(t.e[gi], blockIdx.x - t.first[gi], 0x7fffffffu);
    else limb_gemm_rows_body<NP, false>(t.e[gi], blockIdx.x - t.first[gi], 0x7fffffffu);
}

// ------------------------------------------------------------------ host ---
constexpr size_t kPreferredMost = (size_t)16 << 30;       // of a preferred workspace over Z_2^32
struct Plan {
    int KT, nblkA, nblkB, tilesM, tilesN;
    size_t packA_bytes, packB_bytes;
};
template <class T, class S = GemmShape<T>> inline Plan make_plan(int n, int batch, int M, int N, int K)
{
    Plan p;
    p.KT = ceil_div(K, 32);
    p.tilesM = ceil_div(M, S::BM);
    p.tilesN = ceil_div(N, S::BN);
    p.nblkA = p.tilesM * (S::BM / 32);
    p.nblkB = p.tilesN * (S::BN / 32);
    p.packA_bytes = (size_t)(n + 1) * batch * p.nblkA * p.KT * (S::ND * kFrag);
    p.packB_bytes = (size_t)(n + 1) * batch * p.nblkB * p.KT * (S::ND * kFrag);
    return p;
}
// The tile shapes of a ring: the largest, half of it, and over Z_2^32 a quarter.  The largest takes a CU's registers and LDS, so that
// nothing covers a workgroup's start (3 us), its waits for fragments and its end (3 to 5 us); of the smaller ones two (three over Z_2^32, by quarters)
// share a CU, a tile is done sooner, and more parts of a tile fit the chip.  Half tiles over Z_2^64 have two LDS stages for
// that (three leave a CU one workgroup: 3 % slower in the mean over 6700 products).  Whole calls, full tiles -> the shape taken: 4 parties 224 x 544 x 192 38 ->
// 27 us, 32 x 640 x 2048 60 -> 45, 250 x 301 x 785 41 -> 36; over Z_2^32 2 parties 1024^3 59 -> 47, 3 parties 48 x 3000 x 6000 371 -> 248.
enum TileShape { kFullTile, kHalfTile, kQuarterTile, kShapes };
template <class T> constexpr int shapes_of = Ring<T>::WM * Ring<T>::WN == 4 ? 3 : 2;
template <class T, class F> inline auto with_shape(TileShape shape, F &&fn)
{
    constexpr int WM = Ring<T>::WM, WN = Ring<T>::WN;
    if (shape == kHalfTile) return fn(GemmShape<T, 1, WM * WN / 2>());
    if constexpr (WM * WN == 4)
        if (shape == kQuarterTile) return fn(GemmShape<T, 1, 1>());
    return fn(GemmShape<T>());
}

// The row kernel takes products over Z_2^64 of at most three parties (its units and their LDS) whose inner dimension one launch may accumulate.
inline bool rows_possible(int n, int batch, int M, const Plan &p)
{
    return n <= 3 && p.KT <= Ring<u64>::max_chunk_tiles && rows_grid(batch, M, p.tilesN) <= 0x7fffffffL;
}
constexpr int way_of_shape(TileShape shape) { return SPIN_WAY_FULL_TILES + (int)shape; }

// Estimated times, in microseconds, of a whole call by each kernel: its packs as streams, its launches and its workgroups.  A row item is 2 KT
// half steps (and the waits of the tile that pads an odd KT) and its start and end; its left operands are read once a column tile, from L2 after
// the first, its right fragments once a row block, and where K is odd the rows are loaded word by word.  Outputs of partly filled column tiles
// are stored one by one.  Long calls bring the clock down.  A fit to 4760 products of up to 1.6 times the fastest way's time (1 to 3 parties, 8
// us to 10 ms, sides from 1), within 6.0 % (rms).
inline double row_item_us(int n, int KT) { return (0.1605 + 0.3347 * n) * 2 * KT + 1.217 + 0.352 * n + (KT % 2 ? 0.376 + 0.2475 * n : 0); }
inline double rows_us(int n, int batch, int M, int N, int K, int cus)
{
    const int KT = ceil_div(K, 32), tilesN = ceil_div(N, 64);
    const double rounds = (double)((rows_grid(batch, M, tilesN) + cus - 1) / cus), mb = 16e-6 * n * batch;
    const double left_mb = mb * M * K, right_mb = mb * N * K, out_mb = mb * M * N, written_mb = 8e-6 * (n + 1) * batch * tilesN * 64.0 * KT * 32;
    return 4.72 + 1.805 * n + rounds * row_item_us(n, KT) + 0.051 * n * std::max(0.0, rounds * 2 * KT - 125) + 0.260 * written_mb +
           (0.0454 + (K % 2 ? 0.0367 : 0) + 0.0563 * (tilesN - 1)) * left_mb + 0.1195 * right_mb + (0.0662 + (N % 64 ? 0.0212 : 0)) * out_mb;
}
// The same of the tile kernel by one of its shapes, `splits` workgroups to a tile, each of which adds its part onto Z (the words of Z once more a
// part, and those of C before).  The busiest CU has `most` workgroups; they take their k-steps together as far as its registers and LDS hold several,
// rounds of that many otherwise, and long calls bring the clock down.  Operands are read as they are and written in whole tiles.  Fits to 16 300 timings
// of full and 17 300 of half tiles over Z_2^64 that are within twice the best way's (7 us to 10 ms, 1 to 8 parties, 1 to 16 parts), within 7.0 and 8.4 %
// (rms), and to 91 000, 84 000 and 78 000 over Z_2^32 (5 us to 4 ms, 1 to 6 parties), within 7.1, 8.5 and 9.1 %.  (With the parts' additions
// counted once, 4 parties 192 x 224 x 1504 took 16 parts, not 5: 10 % slower.)
struct TileCost { int at_once; double call, party, round, step, each, start, read, written, out, copied, hot, cool, added, part; };
template <class T> inline const TileCost &tile_cost(TileShape shape)
{
    static constexpr TileCost costs64[] = {{1, 6.74, 1.181, 0.369, 0.906, 0, 3.585, 0.166, 0.223, 0.103, 0.102, 0.274, 34, 0.173, 0},
                                           {2, 6.99, 1.165, 0, 0.6095, 0, 0.368, 0.158, 0.2435, 0.1215, 0.196, 0.2095, 44, 0.131, 0}};
    static constexpr TileCost costs32[] = {{1, 6.73, 0.650, 0.135, 0.552, 0.208, 4.969, 0.013, 0.304, 0.060, 0.127, 0.038, 60, 0.139, 0.026},
                                           {2, 7.76, 0.662, 0.074, 0.309, 0.066, 0.727, 0.000, 0.350, 0.103, 0.110, 0.099, 120, 0.163, 0.031},
                                           {3, 6.98, 0.662, 0.000, 0.215, 0.000, 0.274, 0.000, 0.381, 0.108, 0.170, 0.065, 240, 0.150, 0.038}};
    if constexpr (sizeof(T) == 8) return costs64[shape == kFullTile ? 0 : 1];
    else return costs32[shape];
}
template <class T> struct TileEstimate {
    TileCost c;
    int KT, cus;
    double workgroups, whole_us, out_mb;                 // without parts; all that does not depend on the number of parts
    TileEstimate(int n, int batch, int M, int N, int K, TileShape shape, int cus_) : c(tile_cost<T>(shape)), KT(ceil_div(K, 32)), cus(cus_)
    {
        with_shape<T>(shape, [&](auto s) {
            using S = decltype(s);
            const double tm = ceil_div(M, S::BM), tn = ceil_div(N, S::BN), mb = 1e-6 * sizeof(T) * batch;
            workgroups = tm * tn * n * batch;
            out_mb = 2 * n * mb * (double)M * N;
            whole_us = c.call + c.party * n + c.read * 2 * n * mb * ((double)M + N) * K + c.written * (n + 1) * mb * (tm * S::BM + tn * S::BN) * KT * 32 +
                       c.out * out_mb;
        });
    }
    double us(int splits) const
    {
        const int part = 2 * ceil_div(KT, splits), used = ceil_div(2 * KT, part);
        const double filled = workgroups * used / cus, most = std::ceil(filled);
        return whole_us + part * (c.round * std::floor(filled / c.at_once) + c.step * most + c.each * filled) + c.start * most +
               (used > 1 ? (c.copied + c.added * used) * out_mb + c.part * used : 0) + c.hot * std::max(0.0, most * part - c.cool);
    }
};

// Which digit kernel a product takes, by which tiles, and how many workgroups share one (parts of at least four k-steps): the way that is
// estimated to take the least time.  Over Z_2^32 smaller tiles have to be estimated 6 % faster beyond 60 us, where full ones just fill the chip and
// the estimates are no closer.  Batched products of three parties and one or two k-tiles stay with the row kernel up to 10 % behind: tiles, all packs and
// stores there, take more than estimated (61 entries of 3851 x 83 x 33: 536 us by rows, 624 by half tiles; 257 of 1 x 65 x 2: 40.6 and 44.9).
// Against always the fastest of the digit kernels that costs 0.5 % over 7500 products over Z_2^64 (8 us to 10 ms).
struct DigitRoute { bool rows; int splits; TileShape shape; double us; };
template <class T> inline DigitRoute digit_route(const MatmulArgsT<T> &a, const Plan &p)
{
    const int cus = compute_units();
    DigitRoute r{false, 1, kFullTile, 0};
    double margin = 1, best = 0;
    for (int shape = 0; shape < shapes_of<T>; ++shape) {
        const TileEstimate<T> tiles(a.n, a.batch, a.M, a.N, a.K, (TileShape)shape, cus);
        if (shape == kHalfTile && sizeof(T) == 4 && r.us > 60) margin = 1.06;
        for (int sp = 1; sp <= 16; ++sp) {
            if (sp > 1 && 2 * ceil_div(p.KT, sp) < 4) break;
            if (sp > 1 && ceil_div(p.KT, ceil_div(p.KT, sp)) < sp) continue;         // no more parts than with fewer
            const double us = tiles.us(sp);
            if (best == 0 || margin * us < best) r = DigitRoute{false, sp, (TileShape)shape, us}, best = margin * us;
        }
    }
    if (!std::is_same<T, u64>::value || !rows_possible(a.n, a.batch, a.M, p)) return r;
    const double by_rows = rows_us(a.n, a.batch, a.M, a.N, a.K, cus);
    const bool thin = a.n == 3 && a.batch > 1 && p.KT <= 2;
    if (by_rows <= (thin ? 1.1 : 1) * r.us) r.rows = true, r.us = by_rows;
    return r;
}

// Roughly, for the choice between the digit kernels and the direct one, which takes a product only where this estimate and DigitRoute::us both
// speak for it (alone either of them is off by up to 2.7 times somewhere): 1.5 us a k-step of a full tile (0.85 over Z_2^32), 8 k-steps for start and
// end, as many workgroups to a tile as that makes fastest, and the packs as streams.
template <class T> inline double digit_cost_rough_us(const MatmulArgsT<T> &a, const Plan &p)
{
    const int cus = compute_units();
    const long tiles = (long)p.tilesM * p.tilesN * a.n * a.batch;
    long steps = -1;
    for (int sp = 1; sp <= 16; ++sp) {
        const int part = 2 * ceil_div(p.KT, sp);
        if (sp > 1 && part < 8) break;
        const long cost = (tiles * sp + cus - 1) / cus * (part + 8);
        if (steps < 0 || cost < steps) steps = cost;
    }
    const double pack_bytes = (double)sizeof(T) * (3 * a.n + 1) * a.batch * ((double)a.M + a.N) * a.K;
    const double by_tiles = (sizeof(T) == 8 ? 1.5 : 0.85) * (double)steps + pack_bytes / 5.2e6 + 10;
    if (sizeof(T) != 8 || a.n > 3) return by_tiles;
    return std::min(by_tiles, 1.5 * (double)((rows_grid(a.batch, a.M, p.tilesN) + cus - 1) / cus) * (2 * p.KT + 8) + 10);
}

inline spin_status launch_rows(const MatmulArgs &a, const Plan &p, char *packB, hipStream_t s, const char *where_pack,
                               const char *where_gemm)
{
    launch_pack<u64>(a, nullptr, packB, 0, p.nblkB, p.KT, false, s);
    spin_status st = check_launch(where_pack);
    if (st != SPIN_OK) return st;
    RowGemmArgs g{a.X, a.A, packB, a.C, a.Z, a.batch, a.M, a.N, a.K, p.KT, p.tilesN};
    // One workgroup fits a CU, so more workgroups than CUs only queue: launch one per CU (a multiple of 8, so that
    // an item keeps its XCD) and let each walk its items, its loads running ahead across item boundaries.
    const unsigned items = (unsigned)rows_grid(a.batch, a.M, p.tilesN);
    const unsigned resident = (unsigned)std::max(8, compute_units() / 8 * 8);
    const unsigned grid = items > resident && ((long)items / resident + 1) * p.KT < (1L << 30) ? resident : items;
    for_party_count(a.n, [&](auto np) {
        constexpr int NP = decltype(np)::value <= 3 ? decltype(np)::value : 3;   // n <= 3 is checked by the caller
        auto go = [&](auto vec) {
            static OncePerDevice lds_allowed;
            auto kernel = limb_gemm_rows_kernel<NP, decltype(vec)::value>;
            st = allow_dynamic_lds((const void *)kernel, RowLds<NP>::bytes, lds_allowed);
            if (st != SPIN_OK) return;
            KernelTimer timer(SPIN_KERNEL_GEMM_LIMB, s);
            kernel<<<grid, kRowThreads, RowLds<NP>::bytes, s>>>(g);
            st = check_launch(where_gemm);
        };
        if (a.K % 2 == 0) go(std::true_type());
        else go(std::false_type());
    });
    return st;
}

template <class T, class S>
inline spin_status launch_tiles(const MatmulArgsT<T> &a, int splits, hipStream_t s, const char *where_pack, const char *where_gemm)
{
    const Plan p = make_plan<T, S>(a.n, a.batch, a.M, a.N, a.K);
    char *packA = (char *)a.workspace, *packB = packA + p.packA_bytes;
    const long total = (long)p.tilesM * p.tilesN * a.n * a.batch;
    constexpr int chunk = Ring<T>::max_chunk_tiles;
    // with several workgroups to a tile their parts are added onto Z, which starts out as C
    const bool copy_c = splits > 1 && a.C != a.Z;
    const bool copied = launch_pack<T>(a, packA, packB, p.nblkA, p.nblkB, p.KT, copy_c, s);
    spin_status st = check_launch(where_pack);
    if (st != SPIN_OK) return st;
    if (copy_c && !copied) {
        st = launch_open<T>(a.C, nullptr, (size_t)a.n * a.batch * a.M * a.N, 1, a.Z, s);
        if (st != SPIN_OK) return st;
    }

    static OncePerDevice lds_allowed;                    // one per ring type and shape
    auto kernel = limb_gemm_kernel<T, S>;
    st = allow_dynamic_lds((const void *)kernel, S::lds_bytes, lds_allowed);
    if (st != SPIN_OK) return st;
    GemmArgs<T> g{packA, packB, a.C, a.Z, a.n, a.batch, a.M, a.N, p.nblkA, p.nblkB, p.KT, 0, 0, p.tilesM, p.tilesN,
                  1, 0};
    for (int kt0 = 0; kt0 < p.KT; kt0 += chunk) {
        g.kt0 = kt0;
        g.ktn = p.KT - kt0 < chunk ? p.KT - kt0 : chunk;
        g.C = kt0 == 0 ? a.C : a.Z;                      // later chunks accumulate onto Z
        g.splits = splits;
        g.split_steps = 2 * ceil_div(g.ktn, splits);     // even, so that every part has an even number of steps
        const int used = ceil_div(2 * g.ktn, g.split_steps);     // parts that actually have steps
        g.splits = used;
        if (splits > 1 && used == 1) g.C = a.Z;          // a short last chunk in one part: plain accumulate onto Z
        KernelTimer timer(SPIN_KERNEL_GEMM_LIMB, s);
        kernel<<<(unsigned)(total * used), 256, S::lds_bytes, s>>>(g);
        st = check_launch(where_gemm);
        if (st != SPIN_OK) return st;
    }
    return SPIN_OK;
}

template <class T> spin_status launch_limb(const MatmulArgsT<T> &a, hipStream_t s, const char *where_pack, const char *where_gemm)
{
    const Plan p = make_plan<T>(a.n, a.batch, a.M, a.N, a.K);
    const DigitRoute route = digit_route<T>(a, p);
    if (direct_applies(a.n, a.batch, a.M, a.N, a.K, sizeof(T), digit_cost_rough_us<T>(a, p), route.us))
        return launch_matmul_direct<T>(a, s, where_gemm);
    if constexpr (std::is_same<T, u64>::value) {
        if (ring_macs(a.n, a.batch, a.M, a.N, a.K) >= kResidueMinMacs64) {
            bool taken = false;
            const spin_status st = launch_matmul_residue<T>(a, route.us, s, "spin_beaver_matmul(residue gemm)", taken);
            if (taken) return st;
        }
        if (route.rows) return launch_rows(a, p, (char *)a.workspace + p.packA_bytes, s, where_pack, where_gemm);
    }
    if constexpr (std::is_same<T, u32>::value) {
        bool taken = false;
        const spin_status st = launch_matmul_strassen32(a, s, taken);
        if (taken) return st;
    }

    return with_shape<T>(route.shape, [&](auto shape) { return launch_tiles<T, decltype(shape)>(a, route.splits, s, where_pack, where_gemm); });
}

// ---- grouped call: products of different shapes, a handful of launches for all of them ----------------
// Every group gets its own fragment stores inside the workspace (the packs of all groups run before their
// GEMMs), and the groups share launches: all packs (right operands, and left ones for tiles) in one per kGroupsPerLaunch sides,
// then all GEMMs, by the row or by the tile kernel (grouped_choice), in one per kGroupsPerLaunch groups.  Tiles are not shared between workgroups
// here (the groups together fill the chip), so Z needs no pre-copy.
template <class Args, class Launch> inline void launch_in_tables(const std::vector<Args> &args, const std::vector<unsigned> &blocks, Launch &&launch)
{
    for (size_t g0 = 0; g0 < args.size(); g0 += kGroupsPerLaunch) {
        GroupTable<Args> t;
        t.count = (int)std::min<size_t>(kGroupsPerLaunch, args.size() - g0);
        unsigned total = 0;
        for (int i = 0; i < t.count; ++i) {
            t.first[i] = total;
            t.e[i] = args[g0 + i];
            total += blocks[g0 + i];
        }
        for (int i = t.count; i <= kGroupsPerLaunch; ++i) t.first[i] = total;
        launch(t, total);
    }
}

}  // namespace

struct GroupedWay { bool rows; TileShape shape; };       // rows: with the column tiles of a full tile
static Plan grouped_plan(int n, const MatmulArgs &m, const GroupedWay &w)
{
    return with_shape<u64>(w.rows ? kFullTile : w.shape, [&](auto s) { return make_plan<u64, decltype(s)>(n, m.batch, m.M, m.N, m.K); });
}
// Workgroups of a group's packs and products.
static unsigned long right_pack_blocks(const MatmulArgs &m, const Plan &p)
{
    return (unsigned long)(m.y_transposed ? pack_left_blocks<4>(p.nblkB, p.KT) : pack_right_blocks<4>(p.nblkB, p.KT)) * m.batch;
}
static unsigned long left_pack_blocks(const MatmulArgs &m, const Plan &p) { return (unsigned long)pack_left_blocks<4>(p.nblkA, p.KT) * m.batch; }
static unsigned long grouped_blocks(int n, const MatmulArgs &m, const Plan &p, const GroupedWay &w)
{
    return w.rows ? (unsigned long)rows_grid(m.batch, m.M, p.tilesN) : (unsigned long)p.tilesM * p.tilesN * n * m.batch;
}

// Estimated time in microseconds of a grouped call by the row kernel or by tiles: what its workgroups take of the chip together, the
// longest of them, and the packs as streams.  Fits to 2980 calls of two to twelve products each by rows, full and half tiles (1 to 3 parties, 13 us to 4
// ms; half of them attention products of several stages), within 8.0, 8.2 and 7.7 % (rms).
struct GroupedCost { double call, party, larger, work, longest, read, odd, out, written, hot; };
static double grouped_us(int n, int groups, const MatmulArgs *a, bool by_rows, TileShape shape, int cus)
{
    static constexpr GroupedCost by_row{6.12, 1.376, 0.660, 0.687, 0.188, 0, 0.0356, 0.140, 0.307, 0};
    static constexpr GroupedCost by_tile[2] = {{8.27, 1.222, 0.706, 0.384, 0, 0.1255, 0, 0.0972, 0.261, 0.217},
                                               {7.05, 1.255, 0.746, 0.0644, 0.429, 0.1074, 0, 0.153, 0.300, 0.299}};
    const TileCost &t = tile_cost<u64>(shape);
    const GroupedCost &c = by_rows ? by_row : by_tile[shape];
    double work = 0, longest = 0, streams = 0, steps = 0;
    for (int g = 0; g < groups; ++g) {
        const MatmulArgs &m = a[g];
        const GroupedWay way{by_rows, shape};
        const Plan p = grouped_plan(n, m, way);
        const double each = by_rows ? row_item_us(n, p.KT) : (t.step + t.round) * 2 * p.KT + t.start, mb = 16e-6 * n * m.batch;
        const double share = (double)grouped_blocks(n, m, p, way) / cus;
        work += share * each;
        steps += share * 2 * p.KT;
        longest = std::max(longest, each);
        streams += c.read * mb * ((double)m.M + m.N) * m.K + (m.K % 2 ? c.odd * mb * m.M * m.K : 0) + c.out * mb * m.M * m.N +
                   c.written * 1e-6 * (p.packB_bytes + (by_rows ? 0 : p.packA_bytes));
    }
    return c.call + c.party * n + c.larger * std::max(work, longest) + c.work * work + c.longest * longest + streams + c.hot * std::max(0.0, steps - t.cool);
}

// All products of a call go the same way: the fastest by estimate (the row kernel up to 5 % behind, where the tile estimates are off by more).  Six
// attention products of three stages, by rows and by half tiles: 3 parties 33.6 : 28.4, at twice the batch entries 44.7 : 38.2, at three times 45.9 :
// 48.9, at eight times 110 : 127; 2 parties 26.3 : 28.6, twice 35.6 : 33.3 (and by rows all the same), eight times 74 : 86.  (With the rule for single
// products two of the six went to another launch: 47.8 us.)
static GroupedWay grouped_choice(int n, int groups, const MatmulArgs *a)
{
    const int cus = compute_units();
    const double full = grouped_us(n, groups, a, false, kFullTile, cus), half = grouped_us(n, groups, a, false, kHalfTile, cus);
    const GroupedWay tiles{false, half < full ? kHalfTile : kFullTile};
    for (int g = 0; g < groups; ++g)
        if (!rows_possible(n, a[g].batch, a[g].M, make_plan<u64>(n, a[g].batch, a[g].M, a[g].N, a[g].K))) return tiles;
    return grouped_us(n, groups, a, true, kFullTile, cus) <= 1.05 * std::min(full, half) ? GroupedWay{true, kFullTile} : tiles;
}

// Whether the groups can share launches: not an inner dimension that must be accumulated in several, nor more threads
// than a grid holds (2^32 - 1; a row product's M of 2^24 in 16 batch entries is past it).
static bool grouped_fits(int n, int groups, const MatmulArgs *a, const GroupedWay &w)
{
    unsigned long packs = 0, gemms = 0;
    for (int g = 0; g < groups; ++g) {
        const Plan p = grouped_plan(n, a[g], w);
        if (p.KT > Ring<u64>::max_chunk_tiles) return false;
        packs += right_pack_blocks(a[g], p) + (w.rows ? 0 : left_pack_blocks(a[g], p));
        gemms += grouped_blocks(n, a[g], p, w);
    }
    constexpr unsigned long most = 0xffffffffUL;
    return packs <= most / 256 && gemms <= most / (w.rows ? kRowThreads : 256);
}

// Rows or tiles as estimated, or as asked for; SPIN_EINVAL where that cannot be, SPIN_ERANGE where the groups cannot share launches.
static spin_status grouped_way(int n, int groups, const MatmulArgs *a, const spin_matmul_way *asked, GroupedWay &w)
{
    if (asked == nullptr) {
        w = grouped_choice(n, groups, a);
    } else {
        if (asked->parts != 1 || (asked->kernel != SPIN_WAY_ROWS && asked->kernel != SPIN_WAY_FULL_TILES && asked->kernel != SPIN_WAY_HALF_TILES)) return SPIN_EINVAL;
        w = GroupedWay{asked->kernel == SPIN_WAY_ROWS, asked->kernel == SPIN_WAY_HALF_TILES ? kHalfTile : kFullTile};
        for (int g = 0; g < groups; ++g)
            if (w.rows && !rows_possible(n, a[g].batch, a[g].M, make_plan<u64>(n, a[g].batch, a[g].M, a[g].N, a[g].K))) return SPIN_EINVAL;
    }
    return grouped_fits(n, groups, a, w) ? SPIN_OK : SPIN_ERANGE;
}

spin_matmul_way matmul_grouped_way(int n, int groups, const MatmulArgs *a)
{
    GroupedWay w;
    if (grouped_way(n, groups, a, nullptr, w) != SPIN_OK) return spin_matmul_way{SPIN_WAY_SEPARATE, 1};
    return spin_matmul_way{w.rows ? (int)SPIN_WAY_ROWS : way_of_shape(w.shape), 1};
}

// Returns SPIN_ERANGE, before anything is launched, when the groups cannot share launches; the caller then enqueues
// them one after another.
spin_status launch_matmul_limb_grouped(int n, int groups, const MatmulArgs *a, void *workspace, hipStream_t s, const spin_matmul_way *asked)
{
    GroupedWay way;
    spin_status st = grouped_way(n, groups, a, asked, way);
    if (st != SPIN_OK) return st;
    std::vector<GroupedPackSide> sides;
    std::vector<unsigned> side_blocks, gemm_blocks;
    std::vector<RowGemmArgs> rows;
    std::vector<GemmArgs<u64>> tiles;
    char *ws = (char *)workspace;
    for (int g = 0; g < groups; ++g) {
        const MatmulArgs &m = a[g];
        const Plan p = grouped_plan(n, m, way);
        const int odd = m.K % 2;                         // rows not 16-byte aligned
        char *packA = ws, *packB = ws + p.packA_bytes;
        ws += p.packA_bytes + p.packB_bytes;
        if (m.y_transposed) sides.push_back({PackArgs<u64>{m.Y, m.B, packB, n, m.batch, m.N, m.K, p.nblkB, p.KT}, 2 + odd});
        else sides.push_back({PackArgs<u64>{m.Y, m.B, packB, n, m.batch, m.K, m.N, p.nblkB, p.KT}, 4});
        side_blocks.push_back((unsigned)right_pack_blocks(m, p));
        if (way.rows) {
            rows.push_back(RowGemmArgs{m.X, m.A, packB, m.C, m.Z, m.batch, m.M, m.N, m.K, p.KT, p.tilesN});
        } else {
            sides.push_back({PackArgs<u64>{m.X, m.A, packA, n, m.batch, m.M, m.K, p.nblkA, p.KT}, odd});
            side_blocks.push_back((unsigned)left_pack_blocks(m, p));
            tiles.push_back(GemmArgs<u64>{packA, packB, m.C, m.Z, n, m.batch, m.M, m.N, p.nblkA, p.nblkB, p.KT, 0, p.KT,
                                          p.tilesM, p.tilesN, 1, 2 * p.KT});
        }
        gemm_blocks.push_back((unsigned)grouped_blocks(n, m, p, way));
    }
    for_party_count(n, [&](auto np) {
        constexpr int NP = decltype(np)::value;
        {
            KernelTimer timer(SPIN_KERNEL_PACK, s);
            launch_in_tables(sides, side_blocks, [&](const GroupTable<GroupedPackSide> &t, unsigned total) {
                pack_grouped_kernel<NP><<<total, 256, 0, s>>>(t);
            });
            st = check_launch("spin_beaver_matmul_grouped(pack)");
            if (st != SPIN_OK) return;
        }
        constexpr int RP = NP <= 3 ? NP : 3;                 // groups reach the row kernel only when n <= 3
        if (way.rows) {
            static OncePerDevice lds_allowed;
            auto kernel = limb_gemm_rows_grouped_kernel<RP>;
            st = allow_dynamic_lds((const void *)kernel, RowLds<RP>::bytes, lds_allowed);
            if (st != SPIN_OK) return;
            KernelTimer timer(SPIN_KERNEL_GEMM_LIMB, s);
            launch_in_tables(rows, gemm_blocks, [&](const GroupTable<RowGemmArgs> &t, unsigned total) {
                kernel<<<total, kRowThreads, RowLds<RP>::bytes, s>>>(t);
            });
            st = check_launch("spin_beaver_matmul_grouped(row gemm)");
        } else {
            with_shape<u64>(way.shape, [&](auto sh) {
                using S = decltype(sh);
                static OncePerDevice lds_allowed;
                auto kernel = limb_gemm_grouped_kernel<u64, S>;
                st = allow_dynamic_lds((const void *)kernel, S::lds_bytes, lds_allowed);
                if (st != SPIN_OK) return;
                KernelTimer timer(SPIN_KERNEL_GEMM_LIMB, s);
                launch_in_tables(tiles, gemm_blocks, [&](const GroupTable<GemmArgs<u64>> &t, unsigned total) {
                    kernel<<<total, 256, S::lds_bytes, s>>>(t);
                });
            });
            if (st != SPIN_OK) return;
            st = check_launch("spin_beaver_matmul_grouped(tile gemm)");
        }
    });
    return st;
}

template <class T> spin_matmul_way matmul_way(int n, int batch, int M, int N, int K)
{
    MatmulArgsT<T> a{};
    a.n = n; a.batch = batch; a.M = M; a.N = N; a.K = K;
    const Plan p = make_plan<T>(n, batch, M, N, K);
    const DigitRoute r = digit_route<T>(a, p);
    if (direct_applies(n, batch, M, N, K, sizeof(T), digit_cost_rough_us<T>(a, p), r.us)) return spin_matmul_way{SPIN_WAY_DIRECT, 1};
    return r.rows ? spin_matmul_way{SPIN_WAY_ROWS, 1} : spin_matmul_way{way_of_shape(r.shape), r.splits};
}
template spin_matmul_way matmul_way<u32>(int, int, int, int, int);
template spin_matmul_way matmul_way<u64>(int, int, int, int, int);

template <class T> spin_status launch_matmul_by(const MatmulArgsT<T> &a, const spin_matmul_way &way, hipStream_t s)
{
    constexpr const char *where = "spin_matmul_by";
    const Plan p = make_plan<T>(a.n, a.batch, a.M, a.N, a.K);
    if (way.kernel >= SPIN_WAY_FULL_TILES && way.kernel < SPIN_WAY_FULL_TILES + shapes_of<T>) {
        const int ktn = std::min(p.KT, Ring<T>::max_chunk_tiles);
        if (way.parts < 1 || way.parts > 16 || way.parts > ktn || ceil_div(ktn, ceil_div(ktn, way.parts)) != way.parts) return SPIN_EINVAL;
        return with_shape<T>((TileShape)(way.kernel - SPIN_WAY_FULL_TILES), [&](auto shape) {
            using S = decltype(shape);
            const Plan sp = make_plan<T, S>(a.n, a.batch, a.M, a.N, a.K);
            if ((unsigned long)sp.tilesM * sp.tilesN * a.n * a.batch * way.parts > 0xffffffffUL / 256) return SPIN_ERANGE;
            return launch_tiles<T, S>(a, way.parts, s, where, where);
        });
    }
    if (way.parts != 1) return SPIN_EINVAL;
    if (way.kernel == SPIN_WAY_DIRECT) {
        if ((unsigned long)ceil_div(a.M, 16) * ceil_div(a.N, 16) * a.n * a.batch > 0xffffffffUL / 256) return SPIN_ERANGE;
        return launch_matmul_direct<T>(a, s, where);
    }
    if constexpr (std::is_same<T, u64>::value) {
        if (way.kernel == SPIN_WAY_ROWS)
            return rows_possible(a.n, a.batch, a.M, p) ? launch_rows(a, p, (char *)a.workspace + p.packA_bytes, s, where, where) : SPIN_EINVAL;
        if (way.kernel == SPIN_WAY_RESIDUES) {
            bool taken = false;
            const spin_status st = launch_matmul_residue<T>(a, HUGE_VAL, s, where, taken);
            return taken ? st : SPIN_EWORKSPACE;
        }
    }
    return SPIN_EINVAL;
}
template spin_status launch_matmul_by<u32>(const MatmulArgs32 &, const spin_matmul_way &, hipStream_t);
template spin_status launch_matmul_by<u64>(const MatmulArgs &, const spin_matmul_way &, hipStream_t);

size_t limb_workspace_bytes(int n, int batch, int M, int N, int K)
{
    Plan p = make_plan<u64>(n, batch, M, N, K);
    return p.packA_bytes + p.packB_bytes;
}

size_t limb_preferred_workspace_bytes(int n, int batch, int M, int N, int K)
{
    const Plan p = make_plan<u64>(n, batch, M, N, K);
    if (ring_macs(n, batch, M, N, K) < kResidueMinMacs64) return p.packA_bytes + p.packB_bytes;
    MatmulArgs a{};
    a.n = n; a.batch = batch; a.M = M; a.N = N; a.K = K;
    const size_t need = p.packA_bytes + p.packB_bytes;
    return std::max(need, residue_workspace_bytes<u64>(n, batch, M, N, K, need, digit_route<u64>(a, p).us));
}

size_t limb32_workspace_bytes(int n, int batch, int M, int N, int K)
{
    Plan p = make_plan<u32>(n, batch, M, N, K);
    return p.packA_bytes + p.packB_bytes;
}

size_t limb32_preferred_workspace_bytes(int n, int batch, int M, int N, int K)
{
    return std::max(limb32_workspace_bytes(n, batch, M, N, K), strassen32_workspace_bytes(n, batch, M, N, K, kPreferredMost));
}

spin_status launch_limb32_products(const char *packA, const char *packB, int n, int batch, int M, int N, int K, u32 *Z, hipStream_t s)
{
    using S = GemmShape<u32>;
    static OncePerDevice lds_allowed;
    auto kernel = limb_gemm_kernel<u32>;
    spin_status st = allow_dynamic_lds((const void *)kernel, S::lds_bytes, lds_allowed);
    if (st != SPIN_OK) return st;
    const int KT = K / 32;
    const GemmArgs<u32> g{packA, packB, nullptr, Z, n, batch, M, N, M / 32, N / 32, KT, 0, KT, M / S::BM, N / S::BN, 1, 2 * KT};
    KernelTimer timer(SPIN_KERNEL_GEMM_LIMB, s);
    kernel<<<(unsigned)((long)g.tilesM * g.tilesN * n * batch), 256, S::lds_bytes, s>>>(g);
    return check_launch("spin32_beaver_matmul(limb gemm)");
}

spin_status launch_matmul_limb(const MatmulArgs &a, hipStream_t s)
{
    return launch_limb<u64>(a, s, "spin_beaver_matmul(pack)", "spin_beaver_matmul(limb gemm)");
}

spin_status launch_matmul_limb32(const MatmulArgs32 &a, hipStream_t s)
{
    return launch_limb<u32>(a, s, "spin32_beaver_matmul(pack)", "spin32_beaver_matmul(limb gemm)");
}

}  // namespace spin
