// Strassen's recursion over Z_2^32, two levels above the digit kernels (gemm_limb.hip).
//
// The digit GEMM over Z_2^32 runs at the rate the matrix units sustain on random bytes, so a large product gets faster only by
// fewer multiplications: seven products of half the sides instead of eight (V. Strassen, Gaussian elimination is not optimal,
// 1969).  Sums of blocks wrap like every ring word, so the words are those of the plain product.
//
// Z_i = C_i + E.B_i' + A_i.F: every one of the 49 products P_c takes combination c of the left operands' 16 blocks and
// of the right operands', adds its two operand pairs in one accumulator like any other product, and Z_i is a combination
// of the P_c.  The three passes:
//  strassen_pack_kernel     opens E (F), forms the combinations and stores them as int8 digit fragments, batch entry b of the
//                           call as entries 49 b .. of the GEMM.  Bound by memory: 2n words in, (n + 1) 49/16 out an element (4.4 TB/s).
//  limb_gemm_kernel<u32>    the products, without C.
//  strassen_combine_kernel  Z = C + combinations of the products.
// Measured back to back, whole calls, digit kernels alone against this: two parties 8192^3 16.7 -> 14.8 ms (pack 0.68 -> 1.6, GEMM 15.9 ->
// 12.6, combine 0.53), 6144^3 6.96 -> 6.49, five parties 8192^3 42.9 -> 37.5, three parties 5059 x 7112 x 7399 13.2 -> 11.8.  One
// level alone gains a quarter of it.
#include <algorithm>

#include "limb_common.hpp"

namespace spin {
namespace {

// The combinations: blocks 11, 12, 21, 22 = 0 .. 3; bits 0, 1: first block, 2: it is negative, 3, 4: second block, 5: negative, 6: there is one.
constexpr u32 one(int q) { return (u32)q; }
constexpr u32 sum(int q, int r) { return (u32)q | (u32)r << 3 | 1u << 6; }
constexpr u32 difference(int q, int r) { return sum(q, r) | 1u << 5; }             // q - r
__device__ constexpr u32 kLeftTerms[7] = {sum(0, 3), sum(2, 3), one(0), one(3), sum(0, 1), difference(2, 0), difference(1, 3)};
__device__ constexpr u32 kRightTerms[7] = {sum(0, 3), one(0), difference(1, 3), difference(2, 0), one(3), sum(0, 1), sum(2, 3)};
// kOutput[q][c]: the sign of product c in block q of the result
constexpr int kOutput[4][7] = {{1, 0, 0, 1, -1, 0, 1}, {0, 0, 1, 0, 1, 0, 0}, {0, 1, 0, 1, 0, 0, 0}, {1, -1, 1, 0, 0, 1, 0}};

constexpr int kParts = 4, kBlocks = 16, kProducts = 49;  // parts of a side, blocks of a matrix, products
// block index: the outer quadrant in the high digit (base 4), the inner one in the low; product index: base 7 the same way
__host__ __device__ constexpr int block_row(int q) { return q / 8 * 2 + q / 2 % 2; }
__host__ __device__ constexpr int block_col(int q) { return q / 4 % 2 * 2 + q % 2; }
constexpr int product_sign(int q, int c) { return kOutput[q / 4][c / 7] * kOutput[q % 4][c % 7]; }

struct StrassenSide {
    const u32 *val, *tri;        // X, A or Y, B: [n][batch][rows][cols]
    char *pack;                  // [n+1][batch][49][nblk][KT][4][1024]
    int n, batch, rows, cols;
    int sub_rows, sub_cols;      // of a block (the last ones reach beyond the matrix: zeros)
    int nblk, KT;
};

// One workgroup: the 32 x 32 tiles at one place of all blocks.  A thread loads four elements of each tile; a matrix (a triple share
// as it arrives, then the opened one) goes through LDS, as rows of 32 k whichever side it is, and each wave forms every fourth
// combination of the tiles there: 16 consecutive k a lane, as a fragment wants them.
typedef u32 Unaligned __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kTurnWords = 36;                           // a row of 32 words, 16-byte aligned, off the banks of its neighbours
constexpr int kStrassenLds = kBlocks * 32 * kTurnWords * 4;

template <bool RIGHT, bool VEC>
__global__ __launch_bounds__(256, 2) void strassen_pack_kernel(StrassenSide a)
{
    constexpr int Q = kBlocks;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    u32 *turn = (u32 *)lds;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const unsigned along = RIGHT ? (unsigned)a.nblk : (unsigned)a.KT;      // neighbours read neighbouring columns
    const int major = (int)(blockIdx.x / along), minor = (int)(blockIdx.x % along);
    const int kt = RIGHT ? major : minor, blk = RIGHT ? minor : major, b = blockIdx.z;
    const int row = major * 32 + (int)threadIdx.x / 8, col = minor * 32 + (int)threadIdx.x % 8 * 4;       // within a block
    const size_t mat = (size_t)a.rows * a.cols, party_stride = (size_t)a.batch * mat;
    // An element outside the matrix reads one inside and becomes zero: no load behind a branch.
    auto load = [&](const u32 *base, int q) -> u32x4 {
        const int r = block_row(q) * a.sub_rows + row, c = block_col(q) * a.sub_cols + col;
        const u32 *p = base + (size_t)min(r, a.rows - 1) * a.cols;
        if (VEC) {
            const u32x4 x = __builtin_nontemporal_load((const u32x4 *)(p + min(c, a.cols - 4)));
            return r < a.rows && c < a.cols ? x : (u32x4)(0);
        }
        // Rows that are not 16-byte aligned: the same load at four bytes' alignment, moved to the row's last four elements at its end.
        // (Four loads of an element each: 3.5 times the time of the pack.)
        const int past = max(c - (a.cols - 4), 0);
        const Unaligned y = __builtin_nontemporal_load((const Unaligned *)(p + (c - past)));
        u32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] = 0;
#pragma unroll
            for (int k = 0; e + k < 4; ++k) x[e] = past == k && r < a.rows ? y[e + k] : x[e];
        }
        return x;
    };
    auto emit = [&](const u32x4 (&v)[Q], int slot) {
        __syncthreads();                                 // the combinations of the matrix before are formed
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            u32 *tile = turn + q * (32 * kTurnWords);
            const int r = threadIdx.x / 8, c = threadIdx.x % 8 * 4;
            if (RIGHT) {
#pragma unroll
                for (int e = 0; e < 4; ++e) tile[(c + e) * kTurnWords + r] = v[q][e];
            } else {
                *(u32x4 *)(tile + r * kTurnWords + c) = v[q];
            }
        }
        __syncthreads();
        for (int c = wave; c < kProducts; c += 4) {
            const u32 outer = (RIGHT ? kRightTerms : kLeftTerms)[c / 7];
            const u32 inner = (RIGHT ? kRightTerms : kLeftTerms)[c % 7];
            const u32 *at = turn + lane % 32 * kTurnWords + lane / 32 * 16;
            u32 w[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) w[j] = digit_bias<u32>();
            auto add = [&](int q, bool negative) {
                const u32x4 *p = (const u32x4 *)(at + q * (32 * kTurnWords));
                const u32 flip = negative ? ~0u : 0u;    // -x = ~x + 1
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const u32x4 x = p[j];
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[4 * j + e] += x[e] ^ flip;
                }
                if (negative) {
#pragma unroll
                    for (int j = 0; j < 16; ++j) ++w[j];
                }
            };
            auto inner_terms = [&](int base, bool negative) {
                add(base + (int)(inner & 3), negative);
                if (inner >> 6) add(base + (int)(inner >> 3 & 3), negative != ((inner >> 5 & 1) != 0));
            };
            inner_terms(4 * (int)(outer & 3), false);
            if (outer >> 6) inner_terms(4 * (int)(outer >> 3 & 3), (outer >> 5 & 1) != 0);
#pragma unroll
            for (int j = 0; j < 16; ++j) w[j] ^= digit_bias<u32>();
            store_digit_rows<u32, true>(w, a.pack + (((((size_t)slot * a.batch + b) * kProducts + c) * a.nblk + blk) * a.KT + kt) * (4 * kFrag) +
                                               lane * 16);
        }
    };
    u32x4 opened[Q], v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) opened[q] = (u32x4)(0);
    for (int i = 0; i < a.n; ++i) {
        const size_t at = (size_t)i * party_stride + (size_t)b * mat;
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = load(a.tri + at, q);
#pragma unroll
        for (int q = 0; q < Q; ++q) {                    // eight loads in flight: 16 more would not fit the registers
            opened[q] += load(a.val + at, q) - v[q];
            computed_here(opened[q]);
            if (q % 8 == 7) asm volatile("" ::: "memory");
        }
        if (!RIGHT || i > 0) emit(v, i + 1);
    }
    emit(opened, 0);
    if (RIGHT) {                                         // party 0's slot is B_0 + F
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            opened[q] += load(a.tri + (size_t)b * mat, q);
            computed_here(opened[q]);
            if (q % 8 == 7) asm volatile("" ::: "memory");
        }
        emit(opened, 1);
    }
}

// Four columns of one place of all blocks per thread.  Streams: 49 products and 16 words of C in, 16 words out.
template <bool VEC>
__global__ __launch_bounds__(256) void strassen_combine_kernel(const u32 *products, const u32 *C, u32 *Z, int M, int N, int sub_rows, int sub_cols)
{
    const unsigned quads = (unsigned)sub_cols / 4;
    const unsigned at = blockIdx.x * 256u + threadIdx.x;
    const int r = (int)(at / quads), c = (int)(at % quads) * 4;
    if (r >= sub_rows) return;
    const size_t sub = (size_t)sub_rows * sub_cols, mat = (size_t)M * N;
    const u32 *p = products + blockIdx.y * (kProducts * sub) + (size_t)r * sub_cols + c;
    u32x4 z[kBlocks];
#pragma unroll
    for (int q = 0; q < kBlocks; ++q) z[q] = (u32x4)(0);
#pragma unroll
    for (int k = 0; k < kProducts; ++k) {
        const u32x4 x = __builtin_nontemporal_load((const u32x4 *)(p + k * sub));
#pragma unroll
        for (int q = 0; q < kBlocks; ++q) {
            const int sign = product_sign(q, k);
            if (sign > 0) z[q] += x;
            else if (sign < 0) z[q] -= x;
        }
    }
    const u32 *Cm = C + blockIdx.y * mat;
    u32 *Zm = Z + blockIdx.y * mat;
#pragma unroll
    for (int q = 0; q < kBlocks; ++q) {
        const int row = block_row(q) * sub_rows + r, col = block_col(q) * sub_cols + c;
        if (row >= M) continue;
        const size_t e = (size_t)row * N + col;
        if (VEC) {
            if (col < N) *(u32x4 *)(Zm + e) = *(const u32x4 *)(Cm + e) + z[q];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (col + j < N) Zm[e + j] = Cm[e + j] + z[q][j];
        }
    }
}

// ------------------------------------------------------------------ host ---
struct StrassenPlan {
    bool faster;
    int Ms, Ns, Ks;                                      // sides of a block, whole workgroup tiles
    size_t left_bytes, right_bytes, product_bytes;
    size_t bytes() const { return left_bytes + right_bytes + product_bytes; }
};
inline int part_of(int side, int parts, int multiple) { return ceil_div(ceil_div(side, parts), multiple) * multiple; }

// Rates of both ways: int8 operations on random bytes, bytes of the packs and of the combination, launches.  A fit to 4060 products of 1
// to 8 parties (1 to 4 batch entries, sides of 1024 to 12000, 0.3 to 25 ms), within 4 and 3 % (rms).  647 of them are faster by the
// recursion, 397 by more than 3 %; the rule takes 396, of which 11 are slower by more than 1 %, and costs 0.16 % against always the
// faster way.  (With rates from 30 products it took 8, and cost 0.69 %.)
constexpr double kOpsPerUs = 2.69e9, kPackBytesPerUs = 5.46e6, kCombineBytesPerUs = 2.99e6, kLaunchUs = 66;
constexpr double kPlainOpsPerUs = 2.68e9, kPlainBytesPerUs = 7.16e6, kPlainLaunchUs = 18;

StrassenPlan make_plan(int n, int batch, int M, int N, int K)
{
    StrassenPlan p{};
    // Shorter sides never pay (the blocks' products would have few tiles and k-steps): not worth the estimate.
    if (std::min(std::min(M, N), K) < 1024) return p;
    p.Ms = part_of(M, kParts, 128);
    p.Ns = part_of(N, kParts, 128);
    p.Ks = part_of(K, kParts, 32);
    const double left = (double)p.Ms * p.Ks, right = (double)p.Ks * p.Ns, out = (double)p.Ms * p.Ns;
    const double us = 20.0 * 2 * n * batch * kProducts * out * p.Ks / kOpsPerUs + kLaunchUs +
                      4.0 * batch * (2 * n * kBlocks + (n + 1) * kProducts) * (left + right) / kPackBytesPerUs +
                      4.0 * batch * n * out * (kProducts + 2 * kBlocks) / kCombineBytesPerUs;
    const double m = part_of(M, 1, 128), c = part_of(N, 1, 128), k = part_of(K, 1, 32);
    const double plain_us = 20.0 * 2 * n * batch * m * c * k / kPlainOpsPerUs + 4.0 * batch * (3 * n + 1) * (m * k + k * c) / kPlainBytesPerUs +
                            kPlainLaunchUs;
    const double tiles = (double)n * batch * kProducts * (p.Ms / 128) * (p.Ns / 128);
    const bool fits_grids = (double)n * batch <= 60000 && tiles < 1e9 && (left + right) / 1024 < 1e9 && out / 1024 < 1e9;
    p.faster = us < 0.97 * plain_us && fits_grids;
    p.left_bytes = (size_t)(n + 1) * batch * kProducts * p.Ms * p.Ks * 4;
    p.right_bytes = (size_t)(n + 1) * batch * kProducts * p.Ks * p.Ns * 4;
    p.product_bytes = (size_t)n * batch * kProducts * p.Ms * p.Ns * 4;
    return p;
}

spin_status run(const MatmulArgs32 &a, const StrassenPlan &p, hipStream_t s)
{
    char *left = (char *)a.workspace, *right = left + p.left_bytes, *products = right + p.right_bytes;
    const int KT = p.Ks / 32;
    spin_status st = SPIN_OK;
    {
        KernelTimer timer(SPIN_KERNEL_PACK, s);
        auto go = [&](auto kernel, OncePerDevice &allowed, const StrassenSide &side) {
            st = allow_dynamic_lds((const void *)kernel, kStrassenLds, allowed);
            if (st != SPIN_OK) return;
            kernel<<<dim3((unsigned)(side.nblk * (long)side.KT), 1, a.batch), 256, kStrassenLds, s>>>(side);
            st = check_launch("spin32_beaver_matmul(pack)");
        };
        static OncePerDevice allowed[4];
        const StrassenSide l{a.X, a.A, left, a.n, a.batch, a.M, a.K, p.Ms, p.Ks, p.Ms / 32, KT};
        const StrassenSide r{a.Y, a.B, right, a.n, a.batch, a.K, a.N, p.Ks, p.Ns, p.Ns / 32, KT};
        if (a.K % 4 == 0) go(strassen_pack_kernel<false, true>, allowed[0], l);
        else go(strassen_pack_kernel<false, false>, allowed[1], l);
        if (st != SPIN_OK) return st;
        if (a.N % 4 == 0) go(strassen_pack_kernel<true, true>, allowed[2], r);
        else go(strassen_pack_kernel<true, false>, allowed[3], r);
        if (st != SPIN_OK) return st;
    }
    st = launch_limb32_products(left, right, a.n, a.batch * kProducts, p.Ms, p.Ns, p.Ks, (u32 *)products, s);
    if (st != SPIN_OK) return st;
    KernelTimer timer(SPIN_KERNEL_COMBINE, s);
    const dim3 grid((unsigned)(((long)p.Ms * (p.Ns / 4) + 255) / 256), (unsigned)(a.n * a.batch));
    if (a.N % 4 == 0) strassen_combine_kernel<true><<<grid, 256, 0, s>>>((const u32 *)products, a.C, a.Z, a.M, a.N, p.Ms, p.Ns);
    else strassen_combine_kernel<false><<<grid, 256, 0, s>>>((const u32 *)products, a.C, a.Z, a.M, a.N, p.Ms, p.Ns);
    return check_launch("spin32_beaver_matmul(combine)");
}

}  // namespace

size_t strassen32_workspace_bytes(int n, int batch, int M, int N, int K, size_t most)
{
    const StrassenPlan p = make_plan(n, batch, M, N, K);
    return p.faster && p.bytes() <= most ? p.bytes() : 0;
}

spin_status launch_matmul_strassen32(const MatmulArgs32 &a, hipStream_t s, bool &taken)
{
    const StrassenPlan p = make_plan(a.n, a.batch, a.M, a.N, a.K);
    taken = p.faster && p.bytes() <= a.workspace_bytes;
    return taken ? run(a, p, s) : SPIN_OK;
}

}  // namespace spin
