// Exact ring GEMM over Z_2^128 on the int8 matrix cores (the paper's second ring width: its own
// kernels multiply __int128, Section 6.1).
//
// Same decomposition as the 64-bit kernel with 16 balanced digits: a*b == sum_{i+j<=15} s_i t_j
// 256^(i+j) (mod 2^128), 136 digit pairs on v_mfma_i32_32x32x32_i8, 16 diagonal int32 accumulators,
// result sum_d (int128)D_d << 8d.  D_d needs 128-8d exact bits, so d <= 11 must not overflow:
// 12 * Ktot * 2^14 < 2^31  <=>  Ktot < 10923; for d >= 12 only the low 32 bits matter and wrapping
// leaves them right.  The host splits the inner dimension into chunks of at most 170 k-tiles per
// operand pair (Ktot <= 10880).
//
// Register budget decides the shape: 16 diagonals x 16 accumulator registers fill the 256 AGPRs with
// ONE 32x32 MFMA tile per wave, and the wave's 32 operand fragments (128 VGPRs) cannot be double
// buffered.  So: workgroup tile 64x64 (4 waves as 2x2), two LDS stages of 64 KB, loads of step s+1
// issued between the MFMAs of step s, fragments of a step read at its start.
#include <algorithm>
#include <cmath>

#include "limb_common.hpp"

namespace spin {
namespace {

constexpr int kDigits128 = 16;
constexpr int kMaxChunkTiles128 = 170;    // 2*170*32 = 10880 < 10923 digit products per exact accumulator

struct Gemm128Args {
    const char *packA;   // [n+1][batch][nblkA][KT][16][1024]: slot 0 = E, slot 1+i = A_i
    const char *packB;   // [n+1][batch][nblkB][KT][16][1024]: slot 0 = F, slot 1+i = B_i'
    const u128 *C;       // [n][batch][M][N]  (or Z itself for the later k-chunks)
    u128 *Z;
    int n, batch, M, N;
    int nblkA, nblkB, KT;
    int kt0, ktn;        // this launch covers k-tiles [kt0, kt0+ktn) of both operand pairs
    int tilesM, tilesN;
    int splits, split_steps;     // workgroups per output tile: each takes split_steps of the 2 ktn k-steps and, when splits > 1, adds
};                               // its part onto Z atomically (Z then starts out as C)

struct Shape128 {
    static constexpr int ND = kDigits128;
    static constexpr int NSTAGE = 2;
    static constexpr int BM = 64, BN = 64;                       // 4 waves as 2 x 2, one 32x32 tile each
    static constexpr int FA = BM / 32 * ND, FB = BN / 32 * ND;   // fragments per stage: 32 + 32
    static constexpr int stage_bytes = (FA + FB) * kFrag;        // 64 KB
    static constexpr int lds_bytes = NSTAGE * stage_bytes;
    static constexpr int loads_per_wave = (FA + FB) / 4;         // 16
};

// SPLIT: several workgroups to a tile (with both endings in one kernel it has a register too few).
template <bool SPLIT>
__global__ __launch_bounds__(256) void limb128_gemm_kernel(Gemm128Args g)
{
    using S = Shape128;
    constexpr int ND = S::ND;
    extern __shared__ __attribute__((aligned(1024))) char lds[];

    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int wm = wave / 2, wn = wave % 2;
    // work item = (split, tile), tiles fastest: neighbours on an XCD work on neighbouring tiles of one k-range
    const long tiles_total = (long)g.tilesM * g.tilesN * g.n * g.batch;
    const long item = xcd_contiguous_id(blockIdx.x, tiles_total * g.splits);
    const int split = (int)(item / tiles_total);
    const TileId tile = tile_of(item % tiles_total, g.tilesM, g.tilesN);
    const int pb = tile.pb, tm = tile.tm, tn = tile.tn;
    const int party = pb / g.batch, b = pb % g.batch;

    // fragment streams: step < ktn uses (E, B_i'), step >= ktn uses (A_i, F)
    const size_t blk_stride = (size_t)g.KT * (ND * kFrag);
    const size_t slotA = (size_t)g.batch * g.nblkA * blk_stride;
    const size_t slotB = (size_t)g.batch * g.nblkB * blk_stride;
    const char *a_first = g.packA + (size_t)b * g.nblkA * blk_stride;      // E
    const char *a_second = a_first + (size_t)(1 + party) * slotA;          // A_i
    const char *b_second = g.packB + (size_t)b * g.nblkB * blk_stride;     // F
    const char *b_first = b_second + (size_t)(1 + party) * slotB;          // B_i'

    const int s0 = split * g.split_steps;                // this workgroup's k-steps [s0, s0 + steps)
    const int steps = min(g.split_steps, 2 * g.ktn - s0);
    const bool starts_in_second = s0 >= g.ktn;
    const u32 lds0 = (u32)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const u32 lane16 = lane * 16;

    // Load cursor (scalar unit): this wave loads fragments f = 4q + wave, q < 16: block f / 16 = q / 4
    // of the tile and digit f % 16 = 4 (q % 4) + wave.
    const size_t kt0_off = (size_t)g.kt0 * (ND * kFrag) + wave * kFrag;
    const size_t start_off = (size_t)(starts_in_second ? s0 - g.ktn : s0) * (ND * kFrag) + kt0_off;
    const char *ld_a = (starts_in_second ? a_second : a_first) + (size_t)tm * (S::BM / 32) * blk_stride + start_off;
    const char *ld_b = (starts_in_second ? b_second : b_first) + (size_t)tn * (S::BN / 32) * blk_stride + start_off;
    const char *second_a = a_second + (size_t)tm * (S::BM / 32) * blk_stride + kt0_off;
    const char *second_b = b_second + (size_t)tn * (S::BN / 32) * blk_stride + kt0_off;
    int ld_left = starts_in_second ? 0x7fffffff : g.ktn - s0;            // steps until the cursor switches operand pair
    const u32 ld_lds0 = lds0 + wave * kFrag;
    u32 ld_lds = ld_lds0;
    auto issue_load = [&](int q) {
        constexpr int qa = S::FA / 4, per_blk = ND / 4;
        const char *p = q < qa ? ld_a + (size_t)(q / per_blk) * blk_stride + (q % per_blk) * (4 * kFrag)
                               : ld_b + (size_t)((q - qa) / per_blk) * blk_stride + ((q - qa) % per_blk) * (4 * kFrag);
        load_fragment_to_lds(p, ld_lds + q * (4 * kFrag), lane16);
    };
    auto advance_load_cursor = [&]() {
        ld_a += ND * kFrag;
        ld_b += ND * kFrag;
        if (--ld_left == 0) { ld_a = second_a; ld_b = second_b; }
        ld_lds = ld_lds == ld_lds0 ? ld_lds0 + S::stage_bytes : ld_lds0;     // two stages
    };

    v16i acc[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) acc[d] = (v16i)(0);

    const char *rd_a = lds + (wm * ND) * kFrag + lane16;
    const char *rd_b = lds + (S::FA + wn * ND) * kFrag + lane16;
    int rd_stage = 0;

    // prologue: loads of step 0
#pragma unroll
    for (int q = 0; q < S::loads_per_wave; ++q) issue_load(q);
    advance_load_cursor();

    for (int s = 0; s < steps; ++s) {
        wait_loads<0>();                                 // this wave's loads of step s have landed
        workgroup_barrier();                             // ... everyone's; and every wave is done reading step s-1
        const char *pa = rd_a + rd_stage * S::stage_bytes, *pb_ = rd_b + rd_stage * S::stage_bytes;
        rd_stage ^= 1;
        v4i fa[ND], fb[ND];
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            fb[d] = *(const v4i *)(pb_ + d * kFrag);
            if (d < 2) fa[d] = *(const v4i *)(pa + d * kFrag);
        }
#pragma unroll
        for (int d = 2; d < ND; ++d) fa[d] = *(const v4i *)(pa + d * kFrag);
        __builtin_amdgcn_sched_barrier(0);
        const bool more = s + 1 < steps;
        int slot = 0;
#pragma unroll
        for (int da = 0; da < ND; ++da)
#pragma unroll
            for (int db = 0; db + da < ND; ++db) {
                acc[da + db] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[da], fb[db], acc[da + db], 0, 0, 0);
                // the loads of step s+1 go into the other stage (free since the barrier above), one after
                // every 8th MFMA
                if (slot % 8 == 4 && slot / 8 < S::loads_per_wave) {
                    if (more) issue_load(slot / 8);
                    __builtin_amdgcn_sched_barrier(0);
                }
                ++slot;
            }
        if (more) advance_load_cursor();
    }

    // Recombine the diagonals and add C_i.  All C values are loaded before the first store, so that the
    // loads do not each wait out the store before them (C and Z may be the same buffer); tiles wholly
    // inside the matrix take a branch-free copy, in which the stores do not wait for each other either.
    const size_t mat = (size_t)g.M * g.N;
    const u128 *Cm = g.C + (size_t)pb * mat;
    u128 *Zm = g.Z + (size_t)pb * mat;
    const int col = tn * S::BN + wn * 32 + lane % 32;
    const int row0 = tm * S::BM + wm * 32 + 4 * (lane / 32);
    auto sum_of = [&](int r) {
        u128 v = 0;
#pragma unroll
        for (int d = 0; d < ND; ++d) v += (u128)(__int128)acc[d][r] << (8 * d);
        return v;
    };
    // Parts of a tile: the low words are added first, and the addition that wraps a low word (its return value tells) carries into
    // the high one.  Every wrap is seen by exactly one of the additions, so the sum is right whatever their order.
    if constexpr (SPLIT) {
        u64 low[16], before[16], high[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r / 4) + r % 4;
            const u128 v = sum_of(r);
            low[r] = (u64)v;
            high[r] = (u64)(v >> 64);
            before[r] = 0;
            if (row < g.M && col < g.N)
                before[r] = atomicAdd((unsigned long long *)(Zm + (size_t)row * g.N + col), (unsigned long long)low[r]);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r / 4) + r % 4;
            if (row < g.M && col < g.N)
                atomicAdd((unsigned long long *)(Zm + (size_t)row * g.N + col) + 1, (unsigned long long)(high[r] + (before[r] + low[r] < low[r] ? 1 : 0)));
        }
        return;
    }
    auto epilogue = [&](auto interior_c) {
        constexpr bool INTERIOR = decltype(interior_c)::value;
        u128 cv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r / 4) + r % 4;
            cv[r] = (INTERIOR || (row < g.M && col < g.N)) ? Cm[(size_t)row * g.N + col] : (u128)0;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + 8 * (r / 4) + r % 4;
            const u128 v = cv[r] + sum_of(r);
            if (INTERIOR || (row < g.M && col < g.N)) Zm[(size_t)row * g.N + col] = v;
        }
    };
    if ((tm + 1) * S::BM <= g.M && (tn + 1) * S::BN <= g.N) epilogue(std::true_type());
    else epilogue(std::false_type());
}

struct Plan128 {
    int KT, nblkA, nblkB, tilesM, tilesN;
    size_t packA_bytes, packB_bytes;
};
inline Plan128 make_plan128(int n, int batch, int M, int N, int K)
{
    Plan128 p;
    p.KT = ceil_div(K, 32);
    p.tilesM = ceil_div(M, Shape128::BM);
    p.tilesN = ceil_div(N, Shape128::BN);
    p.nblkA = p.tilesM * (Shape128::BM / 32);
    p.nblkB = p.tilesN * (Shape128::BN / 32);
    p.packA_bytes = (size_t)(n + 1) * batch * p.nblkA * p.KT * (kDigits128 * kFrag);
    p.packB_bytes = (size_t)(n + 1) * batch * p.nblkB * p.KT * (kDigits128 * kFrag);
    return p;
}

// How many workgroups share one output tile (one fits a CU), and the estimated time of the GEMM in microseconds: k-steps (136 MFMAs of
// 32 cycles; faster, at a higher clock, where the tiles leave part of the chip idle), 7.5 us to start and end, and, where parts
// are added onto Z, the copy of C and two atomic additions an element and part; summed over the launches that a long inner
// dimension takes, of which the last is short.  With the pack below a fit to 8700 products of 12 us to 2 ms (1 to 8 parties, 1 to 64
// batch entries, sides 16 to 6500), 5900 of them split, within 7 % (rms) of them and of either kind.  Whole calls, 440 small
// products: 20 % less time than with one workgroup a tile; 4 parties 32 x 32 x 768 135.6 -> 34.0 us, 3 parties 305 x 17 x 875 81.5 -> 38.1.
struct Split128 { int splits, steps; double us; };
inline Split128 choose_splits128(int n, int batch, int M, int N, const Plan128 &p)
{
    const double cus = compute_units(), tiles = (double)p.tilesM * p.tilesN * n * batch, out_mb = 16e-6 * n * batch * (double)M * N;
    const int steps = 2 * std::min(p.KT, kMaxChunkTiles128), full = p.KT / kMaxChunkTiles128, rest = 2 * (p.KT % kMaxChunkTiles128);
    auto launch_us = [&](int chunk_steps, int part) {
        const int used = ceil_div(chunk_steps, part);
        const double filled = tiles * used / cus, rounds = std::ceil(filled);
        return rounds * (3.0 * std::min(part, chunk_steps) * (1 - 0.32 * (1 - filled / rounds)) + 7.5) + (used > 1 ? 0.565 * used * out_mb : 0);
    };
    Split128 best{1, steps, 0};
    for (int want = 1; want <= 16; ++want) {
        const int part = ceil_div(steps, want), used = ceil_div(steps, part);
        if (want > 1 && (part < 2 || used != want)) continue;
        double us = used > 1 ? 1.5 : 0;
        if (full > 0) us += full * launch_us(2 * kMaxChunkTiles128, part);
        if (rest > 0) us += launch_us(rest, part);
        if (want == 1 || us < 0.97 * best.us) best = Split128{used, part, us};
    }
    return best;
}

// Estimated time in microseconds of the pack and this kernel, for the choice against the residue and the direct kernel: the packs as
// streams, and a pack's wave that converts the parties' shares one after another.  Against always taking the fastest of the three
// kernels, on the products above: 0.2 % more time, 3 of them by more than a fifth.  (With the time of one workgroup a tile in its
// place, thin products went to the residue kernels, whose tiles of 256 rows are mostly padding there: 5 parties, two entries of 63
// x 52 x 1950 284 us by residues, 59 by digits; 6.8 % more time over sides of 48 to 2048.)
inline double digit128_cost_us(int n, int batch, int M, int N, int K, const Plan128 &p)
{
    const double pack_bytes = 16.0 * (3 * n + 1) * batch * ((double)M + N) * K;
    return choose_splits128(n, batch, M, N, p).us + pack_bytes / 6.7e6 + 7.4 + 1.55 * n;
}
// The k-steps alone, 3.2 us each: the other side of the direct kernel's own rough estimate.
inline double digit128_rough_us(int n, int batch, const Plan128 &p)
{
    const long tiles = (long)p.tilesM * p.tilesN * n * batch, cus = compute_units();
    return 3.2 * (double)((tiles + cus - 1) / cus) * (2 * p.KT + 4);
}

}  // namespace

size_t limb128_preferred_workspace_bytes(int n, int batch, int M, int N, int K)
{
    const Plan128 p = make_plan128(n, batch, M, N, K);
    if (ring_macs(n, batch, M, N, K) < kResidueMinMacs128) return p.packA_bytes + p.packB_bytes;
    const size_t need = p.packA_bytes + p.packB_bytes;
    return std::max(need, residue_workspace_bytes<u128>(n, batch, M, N, K, need, digit128_cost_us(n, batch, M, N, K, p)));
}

size_t limb128_workspace_bytes(int n, int batch, int M, int N, int K)
{
    Plan128 p = make_plan128(n, batch, M, N, K);
    return p.packA_bytes + p.packB_bytes;
}

spin_status launch_matmul_limb128(const MatmulArgs128 &a, hipStream_t s)
{
    const Plan128 p = make_plan128(a.n, a.batch, a.M, a.N, a.K);
    const double digits_us = digit128_cost_us(a.n, a.batch, a.M, a.N, a.K, p);
    if (direct_applies(a.n, a.batch, a.M, a.N, a.K, 16, digit128_rough_us(a.n, a.batch, p), digits_us)) return launch_matmul_direct<u128>(a, s, "spin128_beaver_matmul(direct)");
    spin_status st = SPIN_OK;
    if (ring_macs(a.n, a.batch, a.M, a.N, a.K) >= kResidueMinMacs128) {
        bool taken = false;
        st = launch_matmul_residue<u128>(a, digits_us, s, "spin128_beaver_matmul(residue gemm)", taken);
        if (taken) return st;
    }
    char *packA = (char *)a.workspace;
    char *packB = packA + p.packA_bytes;
    const Split128 split = choose_splits128(a.n, a.batch, a.M, a.N, p);
    // with several workgroups to a tile their parts are added onto Z, which starts out as C
    const bool copy_c = split.splits > 1 && a.C != a.Z;
    const bool copied = launch_pack<u128>(a, packA, packB, p.nblkA, p.nblkB, p.KT, copy_c, s);
    st = check_launch("spin128_beaver_matmul(pack)");
    if (st != SPIN_OK) return st;
    if (copy_c && !copied) {
        st = launch_open<u128>(a.C, nullptr, (size_t)a.n * a.batch * a.M * a.N, 1, a.Z, s);
        if (st != SPIN_OK) return st;
    }

    static OncePerDevice lds_allowed[2];
    auto launch = [&](auto kernel, OncePerDevice &allowed, const Gemm128Args &g, long workgroups) {
        st = allow_dynamic_lds((const void *)kernel, Shape128::lds_bytes, allowed);
        if (st != SPIN_OK) return;
        KernelTimer timer(SPIN_KERNEL_GEMM_LIMB, s);
        kernel<<<(unsigned)workgroups, 256, Shape128::lds_bytes, s>>>(g);
        st = check_launch("spin128_beaver_matmul(limb gemm)");
    };
    Gemm128Args g{packA, packB, a.C, a.Z, a.n, a.batch, a.M, a.N, p.nblkA, p.nblkB, p.KT, 0, 0, p.tilesM, p.tilesN,
                  1, split.steps};
    const long total = (long)p.tilesM * p.tilesN * a.n * a.batch;
    for (int kt0 = 0; kt0 < p.KT; kt0 += kMaxChunkTiles128) {
        g.kt0 = kt0;
        g.ktn = p.KT - kt0 < kMaxChunkTiles128 ? p.KT - kt0 : kMaxChunkTiles128;
        g.C = kt0 == 0 && split.splits == 1 ? a.C : a.Z; // later chunks, and parts, accumulate onto Z
        g.splits = ceil_div(2 * g.ktn, split.steps);     // parts that have steps (a short last chunk may need one, as a plain addition)
        if (g.splits > 1) launch(limb128_gemm_kernel<true>, lds_allowed[1], g, total * g.splits);
        else launch(limb128_gemm_kernel<false>, lds_allowed[0], g, total);
        if (st != SPIN_OK) return st;
    }
    return SPIN_OK;
}

}  // namespace spin
