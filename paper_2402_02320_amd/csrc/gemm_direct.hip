// The Beaver matmul of small products in one launch: no pack, no workspace.  A 64^3 product of three parties is 1.6e6
// ring multiply-adds, a microsecond of vector arithmetic, but the limb path spends 6.6 us on packing its right operand
// and 12.7 us on a GEMM of two workgroups.  Here a workgroup owns a 16 x 16 tile of one party's output, opens its own
// 16 rows of E and 16 columns of F (again in every tile: the operands come from L2) and multiplies on the vector ALU.
//
// What bounds it: per tile and 64 k, 4 n x 16 x 64 words are fetched (98 KB for three parties, about 10 ns of the chip's
// L2 bandwidth) for 32768 multiply-adds (4 ns of its vector rate); so it is the faster one only while its few
// microseconds of latency and that traffic stay below the limb path's fixed cost (direct_applies).
#include "limb_common.hpp"

namespace spin {
namespace {

constexpr int kTile = 16;
// inner dimension per round: four operand tiles of 8448 bytes in LDS (4352 of 4-byte elements), up to four workgroups to a CU
template <class T> constexpr int kDepth = sizeof(T) == 16 ? 32 : 64;

template <class T> struct DirectArgs {
    const T *X, *Y, *A, *B, *C;
    T *Z;
    int batch, M, N, K;
    int tilesM, tilesN;
    bool y_transposed;
};

template <class T, int NP>
__global__ __launch_bounds__(256) void direct_matmul_kernel(DirectArgs<T> g)
{
    constexpr int KD = kDepth<T>, kPitch = KD + 16 / (int)sizeof(T);     // rows a 16-byte bank group apart
    constexpr int kEach = kTile * KD / 256;                              // elements of a tile that one thread loads
    __shared__ __attribute__((aligned(16))) T tile[4][kTile * kPitch];   // E, A_p [row][k]; B_p', F [column][k]
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    unsigned id = blockIdx.x;
    const int tn = (int)(id % (unsigned)g.tilesN);
    id /= (unsigned)g.tilesN;
    const int tm = (int)(id % (unsigned)g.tilesM);
    id /= (unsigned)g.tilesM;
    const int b = (int)(id % (unsigned)g.batch), party = (int)(id / (unsigned)g.batch);
    const size_t xmat = (size_t)g.M * g.K, ymat = (size_t)g.K * g.N, zmat = (size_t)g.M * g.N;
    const T *X = g.X + b * xmat, *A = g.A + b * xmat, *Y = g.Y + b * ymat, *B = g.B + b * ymat;
    const size_t xstride = g.batch * xmat, ystride = g.batch * ymat;
    const int row0 = tm * kTile, col0 = tn * kTile;

    // wave w multiplies the w-th quarter of every round's k; a lane owns 2 x 2 outputs
    T acc[2][2] = {};
    const int r2 = lane / 8 * 2, c2 = lane % 8 * 2;
    for (int k0 = 0; k0 < g.K; k0 += KD) {
        // Loads are unconditional: rows, columns and k beyond the matrix read its last ones.  What rows and columns bring
        // is never stored; for k >= K the left values are zeroed.
        T e[kEach], a[kEach], f[kEach], bp[kEach];
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int i = tid + 256 * j;
            const int lk = i % KD, lr = i / KD;
            const size_t left = (size_t)min(row0 + lr, g.M - 1) * g.K + min(k0 + lk, g.K - 1);
            const int rk = g.y_transposed ? i % KD : i / kTile, rc = g.y_transposed ? i / KD : i % kTile;
            const size_t ck = min(k0 + rk, g.K - 1), cc = min(col0 + rc, g.N - 1);
            const size_t right = g.y_transposed ? cc * g.K + ck : ck * g.N + cc;
            e[j] = f[j] = 0;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const T av = A[p * xstride + left], bv = B[p * ystride + right];
                e[j] += X[p * xstride + left] - av;
                f[j] += Y[p * ystride + right] - bv;
                a[j] = p == 0 || p == party ? av : a[j];
                bp[j] = p == 0 || p == party ? bv : bp[j];
            }
        }
        if (k0 > 0) __syncthreads();                     // the previous round is read
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int i = tid + 256 * j;
            const int lk = i % KD, lr = i / KD;
            const bool ok = k0 + lk < g.K;
            tile[0][lr * kPitch + lk] = ok ? e[j] : (T)0;
            tile[1][lr * kPitch + lk] = ok ? a[j] : (T)0;
            const int rk = g.y_transposed ? i % KD : i / kTile, rc = g.y_transposed ? i / KD : i % kTile;
            tile[2][rc * kPitch + rk] = party == 0 ? bp[j] + f[j] : bp[j];
            tile[3][rc * kPitch + rk] = f[j];
        }
        __syncthreads();
#pragma unroll 4
        for (int k = wave * (KD / 4); k < (wave + 1) * (KD / 4); ++k) {
            T ev[2], av[2], bv[2], fv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                ev[i] = tile[0][(r2 + i) * kPitch + k];
                av[i] = tile[1][(r2 + i) * kPitch + k];
                bv[i] = tile[2][(c2 + i) * kPitch + k];
                fv[i] = tile[3][(c2 + i) * kPitch + k];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] += ev[i] * bv[j] + av[i] * fv[j];
        }
    }
    __syncthreads();
    T *part = &tile[0][0];                               // [wave][16][16]: 4 x 256 elements over the first one or two tiles
    static_assert(4 * 256 <= 4 * kTile * kPitch, "the partial sums fit the tiles");
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) part[wave * 256 + (r2 + i) * kTile + c2 + j] = acc[i][j];
    __syncthreads();
    const int row = row0 + tid / kTile, col = col0 + tid % kTile;
    if (row < g.M && col < g.N) {
        const size_t at = ((size_t)party * g.batch + b) * zmat + (size_t)row * g.N + col;
        g.Z[at] = g.C[at] + part[tid] + part[256 + tid] + part[512 + tid] + part[768 + tid];
    }
}

}  // namespace

// Estimated time against that of the digit kernels, twice; both have to speak for this kernel.
//
// Roughly: a workgroup's round (load, open, multiply) takes 1.45, 2.8 or 4.2 us over 4-, 8- or 16-byte elements however few tiles
// there are; beyond that a tile costs the chip 2 or 8 ns for three parties.  The rough digit estimate is about a third high for
// the smallest products, hence the factors.
//
// In detail: a round's latency grows with the parties, tiles share the chip, and a k-slab of operands that outgrows an XCD's L2 (4
// MB) has to be read anew by every tile that wants it.  Fits to 12 500 products that the rough estimate takes, within 10 % (rms), and
// 7 to 10 % on the digit side.  Out of 22 000 products near the line the rough estimate alone takes these by more than 2 % wrongly:
// 352 over Z_2^32 (up to 2.8 times: 5 parties, batch 61, 6 x 943 x 228, 1014 us against 362), 77 over Z_2^64 (1.8 times: 7 parties,
// batch 19, 13 x 476 x 43, 135 against 74), 10 over Z_2^128; wide and batched products above all.  With both it is 76, 45 and 2.  The line lies 3 % to the side of the digit kernels
// over Z_2^32 and Z_2^128 and 2 % to this one's over Z_2^64, whose digit estimates are later ones: 7470 products there, this kernel among the ways,
// cost 0.63 % against always the fastest (0.69 at a line of 0.97).
//
// Measured, this against the limb path: 3 parties 64^3 5.7 : 18.8 us, 128^3 9.7 : 23.8, 256 x 256 x 64 10.4 : 19.6; left to the limb
// path: 256^3 30.9 : 25.4, 2 parties 64 x 64 x 512 24.8 : 21.9, 3 parties 512 x 512 x 32 29.2 : 17.7.  Over Z_2^128 long inner
// dimensions are the residue GEMM's.
bool direct_applies(int n, int batch, int M, int N, int K, int elem_bytes, double rough_us, double digits_us)
{
    const int tilesM = ceil_div(M, kTile), tilesN = ceil_div(N, kTile);
    const double tiles = (double)tilesM * tilesN * n * batch;
    const int rounds = ceil_div(K, elem_bytes == 16 ? kDepth<u128> : kDepth<u64>);
    const double each = (elem_bytes == 4 ? 0.002 : 0.008) * (n + 1) / 4;
    const double base = elem_bytes == 4 ? 1.45 : elem_bytes == 8 ? 2.8 : 4.2;
    if (elem_bytes == 16 && rounds > 8) return false;
    if (2.5 + rounds * (base + each * tiles) >= (elem_bytes == 16 ? 0.75 : 0.62) * rough_us) return false;

    struct Cost { double launch, round, round_party, share, share_party, slab_mb, mb_per_us, alone; };
    // alone: how much more of the chip a tile takes where the registers leave a CU one workgroup (7 and 8 parties over Z_2^64, 4 to 8
    // over Z_2^128)
    const Cost c = elem_bytes == 4   ? Cost{2.24, 1.00, 0.106, 0.458, 0.148, 1.85, 27.4, 0}
                   : elem_bytes == 8 ? Cost{2.13, 1.81, 0.371, 0.984, 0.313, 2.04, 29.2, n >= 7 ? 0.366 : 0}
                                     : Cost{2.42, 3.55, 0.160, 1.855, 0.153, 1.98, 20.0, n >= 4 ? 0.844 : 0};
    const double w = elem_bytes, slab_mb = 2.0 * n * batch * ((double)M + N) * K * w / rounds / 1e6;
    // bytes of one row of a right operand's tile, in whole lines where its neighbours have the rest of them
    const double row = tilesN == 1 ? N * w : kTile * w + (N * elem_bytes % 128 == 0 ? 0 : 64);
    const double read_mb = 2.0 * n * K * (tiles * row + (double)tilesN * n * batch * M * w) / 1e6;
    const double missed = slab_mb > c.slab_mb ? 1 - c.slab_mb / slab_mb : 0;
    const double us = c.launch + rounds * (c.round + c.round_party * n + (c.share + c.share_party * n) * (1 + c.alone) * tiles / 256) +
                      missed * read_mb / c.mb_per_us;
    return us < (elem_bytes == 8 ? 1.02 : 0.97) * digits_us;
}

template <class T> spin_status launch_matmul_direct(const MatmulArgsT<T> &a, hipStream_t s, const char *where)
{
    DirectArgs<T> g{a.X, a.Y, a.A, a.B, a.C, a.Z, a.batch, a.M, a.N, a.K, ceil_div(a.M, kTile), ceil_div(a.N, kTile), a.y_transposed};
    const unsigned blocks = (unsigned)((long)g.tilesM * g.tilesN * a.n * a.batch);
    KernelTimer timer(SPIN_KERNEL_GEMM_DIRECT, s);
    for_party_count(a.n, [&](auto np) { direct_matmul_kernel<T, decltype(np)::value><<<blocks, 256, 0, s>>>(g); });
    return check_launch(where);
}
template spin_status launch_matmul_direct<u32>(const MatmulArgsT<u32> &, hipStream_t, const char *);
template spin_status launch_matmul_direct<u64>(const MatmulArgsT<u64> &, hipStream_t, const char *);
template spin_status launch_matmul_direct<u128>(const MatmulArgsT<u128> &, hipStream_t, const char *);

}  // namespace spin
