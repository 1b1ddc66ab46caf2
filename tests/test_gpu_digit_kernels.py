"""The digit kernels at the sizes where they can go wrong, against the CPU oracle: edges of their 32-wide blocks and 64- and
128-wide tiles, of their k-tiles and of the k-tiles that a row item walks, every party count, batches, transposed right operands, C
updated in place.  The products are such that the library gives them to these kernels (most small ones go to the one-launch kernel,
large ones to the residue GEMM): the kernel class that it reports is checked.  Which of the digit kernels takes a product is the
library's choice; the row kernel is asked for by name as well wherever it can be.  Exact ring words."""
import numpy as np
import pytest
import torch

import oracle
from oracle import r128
from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu

# n, batch, M, N, K
ROWS = [(2, 2, 200, 257, 160), (2, 32, 192, 1, 226), (1, 32, 130, 64, 192), (3, 32, 1, 65, 226), (2, 12, 65, 129, 66),
        (3, 4, 65, 200, 96), (3, 6, 192, 64, 96), (1, 12, 257, 65, 160), (3, 12, 129, 31, 226), (3, 48, 32, 63, 512),
        (2, 48, 2, 127, 1500), (3, 16, 130, 63, 34), (3, 16, 1, 130, 512), (2, 3, 257, 129, 192), (2, 48, 1, 128, 226),
        (3, 128, 1, 65, 34), (3, 32, 63, 31, 700), (1, 64, 63, 96, 512), (1, 24, 96, 127, 226), (3, 6, 128, 257, 258),
        (2, 12, 192, 65, 512), (3, 6, 128, 192, 2), (3, 24, 127, 33, 64), (2, 16, 127, 63, 192), (3, 64, 2, 64, 1000),
        (3, 4, 192, 64, 258), (2, 64, 1, 128, 1500), (2, 48, 64, 96, 32), (2, 32, 32, 127, 66), (3, 32, 32, 128, 2),
        (3, 16, 130, 31, 1000), (3, 12, 192, 63, 32), (3, 8, 32, 192, 160), (3, 6, 127, 96, 258), (3, 2, 128, 200, 160),
        (3, 6, 128, 65, 160), (2, 128, 2, 128, 34), (3, 48, 1, 127, 128), (2, 16, 257, 33, 32), (1, 96, 2, 128, 1500),
        (3, 16, 64, 63, 96), (2, 128, 63, 2, 66), (3, 64, 192, 1, 2), (1, 12, 128, 200, 66)]
TILES = [(4, 1, 128, 257, 258), (4, 1, 192, 128, 700), (5, 48, 65, 2, 31), (6, 6, 63, 64, 96), (5, 3, 127, 129, 34),
         (8, 1, 31, 32, 1500), (7, 6, 63, 33, 95), (7, 4, 64, 2, 258), (7, 1, 129, 130, 512), (2, 128, 96, 31, 33),
         (2, 24, 200, 65, 160), (7, 2, 130, 63, 97), (8, 2, 33, 257, 64), (2, 16, 192, 192, 32), (5, 3, 96, 65, 160),
         (1, 1, 64, 200, 1000), (4, 12, 63, 127, 33), (4, 1, 96, 127, 1000), (5, 1, 200, 63, 700), (6, 1, 257, 192, 32),
         (4, 6, 130, 64, 96), (2, 1, 1, 32, 1000), (1, 96, 127, 33, 31), (6, 1, 127, 192, 512), (6, 24, 128, 1, 32),
         (8, 1, 200, 129, 96), (7, 1, 128, 257, 32), (7, 1, 130, 64, 700), (1, 96, 96, 64, 226), (7, 1, 127, 63, 226),
         (4, 16, 129, 1, 160), (7, 1, 130, 128, 1500), (2, 16, 257, 65, 96), (1, 48, 192, 33, 160), (5, 1, 63, 31, 1500),
         (1, 32, 129, 96, 192), (5, 3, 33, 200, 95), (8, 1, 63, 200, 512), (5, 8, 64, 64, 66), (6, 12, 96, 31, 31),
         (6, 16, 200, 2, 34), (5, 1, 96, 129, 1500), (8, 1, 96, 128, 66), (5, 32, 64, 31, 34)]
TILES32 = [(8, 3, 33, 96, 226), (3, 48, 33, 33, 226), (6, 3, 127, 130, 66), (2, 64, 64, 127, 31), (2, 32, 65, 130, 97),
           (8, 32, 32, 63, 2), (8, 2, 200, 128, 95), (7, 8, 63, 65, 66), (5, 6, 200, 130, 64), (8, 1, 96, 128, 258),
           (7, 4, 127, 64, 160), (7, 1, 33, 2, 1000), (7, 24, 96, 33, 31), (8, 32, 127, 1, 2), (1, 64, 257, 33, 95),
           (4, 6, 200, 130, 97), (5, 12, 96, 65, 66), (1, 96, 63, 129, 192), (1, 1, 129, 192, 700), (4, 16, 192, 31, 95),
           (2, 96, 96, 63, 32), (3, 12, 130, 200, 1), (1, 128, 96, 128, 33), (5, 24, 130, 32, 96), (2, 1, 192, 65, 512),
           (4, 1, 128, 128, 512), (7, 12, 257, 32, 33), (8, 64, 1, 127, 34), (4, 1, 129, 130, 512), (6, 12, 32, 192, 128)]
TILES128 = [(3, 64, 31, 2, 96), (6, 1, 192, 127, 97), (1, 128, 32, 33, 97), (6, 2, 128, 31, 226), (7, 24, 31, 2, 33),
            (1, 8, 257, 96, 66), (6, 1, 129, 129, 160), (3, 48, 1, 33, 95), (4, 24, 33, 32, 34), (7, 1, 2, 32, 700),
            (5, 8, 32, 64, 95), (2, 96, 31, 31, 64), (3, 1, 192, 1, 1000), (6, 1, 257, 127, 66), (4, 1, 257, 65, 192),
            (8, 1, 129, 64, 258), (2, 6, 96, 192, 64), (1, 16, 130, 257, 31), (7, 2, 192, 2, 128), (8, 6, 1, 64, 96),
            (1, 1, 32, 127, 512), (7, 1, 127, 200, 96), (3, 2, 200, 33, 700), (3, 16, 96, 1, 192), (1, 6, 129, 192, 160),
            (1, 8, 130, 96, 226)]


def by_digits(f):
    """f's result, and that the digit kernels made it."""
    spin.profile_reset()
    spin.profile_enable(True)
    out = f()
    torch.cuda.synchronize()
    spin.profile_enable(False)
    count = {k: spin.profile_read(k)[1] for k in ("gemm_limb", "gemm_direct", "gemm_residue")}
    spin.profile_reset()
    assert count["gemm_limb"] > 0 and count["gemm_direct"] == count["gemm_residue"] == 0, "goes to another kernel now: %s" % count
    return out


def dev(a, dtype=np.int64):
    return torch.from_numpy(np.ascontiguousarray(a).view(dtype)).cuda()


def host(t, dtype=np.uint64):
    return t.cpu().numpy().view(dtype)


def draw(n, batch, M, N, K, bits=64):
    rng = np.random.default_rng(M * 1000 + N * 10 + K)
    w = (2,) if bits == 128 else ()
    top = 1 << min(bits, 64)
    X = rng.integers(0, top, size=(n, batch, M, K) + w, dtype=np.uint64)
    Y = rng.integers(0, top, size=(n, batch, K, N) + w, dtype=np.uint64)
    deal = r128.dealer_matmul if bits == 128 else oracle.dealer_matmul
    return (X, Y) + tuple(deal(n, batch, M, N, K, seed=K, **({"l": 32} if bits == 32 else {})))


@pytest.mark.parametrize("n,batch,M,N,K", ROWS + TILES)
def test_ring64(n, batch, M, N, K):
    X, Y, A, B, C = draw(n, batch, M, N, K)
    want = oracle.beaver_matmul(X, Y, A, B, C)
    ops = [dev(t) for t in (X, Y, A, B, C)]
    assert (host(by_digits(lambda: spin.beaver_matmul(*ops))) == want).all()
    Yt, Bt = (dev(t.transpose(0, 1, 3, 2)) for t in (Y, B))
    if n <= 3:
        assert (host(spin.beaver_matmul_by("rows", 1, *ops)) == want).all()
        assert (host(spin.beaver_matmul_by("rows", 1, ops[0], Yt, ops[2], Bt, ops[4], y_transposed=True)) == want).all()
    assert (host(by_digits(lambda: spin.beaver_matmul(ops[0], Yt, ops[2], Bt, ops[4], y_transposed=True))) == want).all()
    assert (host(ops[4]) == C).all()
    by_digits(lambda: spin.beaver_matmul(*ops, out=ops[4]))
    assert (host(ops[4]) == want).all()


@pytest.mark.parametrize("n,batch,M,N,K", TILES32)
def test_ring32(n, batch, M, N, K):
    X, Y, A, B, C = draw(n, batch, M, N, K, 32)
    want = oracle.beaver_matmul(X, Y, A, B, C, l=32)
    ops = [dev(t.astype(np.uint32), np.int32) for t in (X, Y, A, B, C)]
    assert (host(by_digits(lambda: spin.ring32.beaver_matmul(*ops)), np.uint32) == want).all()
    by_digits(lambda: spin.ring32.beaver_matmul(*ops, out=ops[4]))
    assert (host(ops[4], np.uint32) == want).all()


# 16 x 16 outputs: below the products for which residues are considered, so the inner dimension may pass the 170 k-tiles of one chunk
@pytest.mark.parametrize("n,batch,M,N,K", TILES128 + [(2, 1, 16, 16, 170 * 32), (2, 1, 16, 16, 170 * 32 + 1), (3, 1, 15, 9, 2 * 170 * 32 + 31)])
def test_ring128(n, batch, M, N, K):
    X, Y, A, B, C = draw(n, batch, M, N, K, 128)
    want = r128.beaver_matmul(X, Y, A, B, C)
    ops = [dev(t) for t in (X, Y, A, B, C)]
    assert (host(by_digits(lambda: spin.ring128.beaver_matmul(*ops))) == want).all()
    by_digits(lambda: spin.ring128.beaver_matmul(*ops, out=ops[4]))
    assert (host(ops[4]) == want).all()


def test_ring128_worst_case_digits_over_two_chunks():
    # all sixteen digits of E, F, A_1 and B_1 equal to -128: the int32 sums of a chunk at their extreme
    n, M, N, K = 2, 16, 16, 170 * 32 + 64
    worst = np.array([0x7F7F7F7F7F7F7F80, 0x7F7F7F7F7F7F7F7F], dtype=np.uint64)
    X, Y = np.zeros((n, 1, M, K, 2), dtype=np.uint64), np.zeros((n, 1, K, N, 2), dtype=np.uint64)
    A, B, C = np.zeros_like(X), np.zeros_like(Y), np.zeros((n, 1, M, N, 2), dtype=np.uint64)
    X[:], Y[:], A[1], B[1] = worst, worst, worst, worst
    got = by_digits(lambda: spin.ring128.beaver_matmul(*(dev(t) for t in (X, Y, A, B, C))))
    assert (host(got) == r128.beaver_matmul(X, Y, A, B, C)).all()


@pytest.mark.parametrize("M,K", [(4200, 511 * 32), (300, 511 * 32), (32, 511 * 32 + 96)])
def test_ring64_worst_case_digits(M, K):
    # all digits -128 over the longest inner dimension that is accumulated at once, few tiles and many, and a second chunk (by the library's choice;
    # each kernel by its name: test_gpu_named_kernels.py)
    n, N = 2, 64
    worst = torch.tensor(0x7F7F7F7F7F7F7F80, dtype=torch.int64, device="cuda")
    X, Y = worst.expand(n, 1, M, K).contiguous(), worst.expand(n, 1, K, N).contiguous()
    A, B = torch.zeros_like(X), torch.zeros_like(Y)
    A[1], B[1] = worst, worst
    C = torch.zeros(n, 1, M, N, dtype=torch.int64, device="cuda")
    got = by_digits(lambda: spin.beaver_matmul(X, Y, A, B, C))
    w, m = 0x7F7F7F7F7F7F7F80, 1 << 64
    for i in range(n):                                   # E = F = worst; Z_0 = E (B_0 + F) + A_0 F, Z_1 = E B_1 + A_1 F
        v = (1 if i == 0 else 2) * K * w * w % m
        assert bool((got[i] == (v - m if v >> 63 else v)).all())
