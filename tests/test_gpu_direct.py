"""The one-launch kernel of small Beaver matmuls against the CPU oracle: sizes around its 16 x 16 tile and its 64-deep (32
over Z_2^128) round, every party count, batches, transposed right operands, C updated in place.  Ring words, so equality is
exact.  The shapes are ones its rule takes: the kernel class that the library reports having launched is checked."""
import numpy as np
import pytest
import torch

import oracle
from oracle import r128
from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu

SHAPES = [(3, 1, 64, 64, 64), (1, 1, 1, 1, 1), (2, 1, 16, 16, 64), (5, 1, 17, 15, 65), (8, 1, 31, 33, 63), (2, 3, 48, 20, 128),
          (4, 2, 16, 1, 129), (3, 1, 1, 200, 31), (6, 1, 100, 17, 64), (7, 1, 33, 33, 2)]


def launched_direct(f):
    spin.profile_reset()
    spin.profile_enable(True)
    out = f()
    torch.cuda.synchronize()
    spin.profile_enable(False)
    count = spin.profile_read("gemm_direct")[1]
    spin.profile_reset()
    return out, count == 1


def dev(a, dtype=np.int64):
    return torch.from_numpy(np.ascontiguousarray(a).view(dtype)).cuda()


@pytest.mark.parametrize("n,batch,M,N,K", SHAPES)
def test_ring64(n, batch, M, N, K):
    rng = np.random.default_rng(M * 1000 + K)
    X = rng.integers(0, 1 << 64, size=(n, batch, M, K), dtype=np.uint64)
    Y = rng.integers(0, 1 << 64, size=(n, batch, K, N), dtype=np.uint64)
    A, B, C = oracle.dealer_matmul(n, batch, M, N, K, seed=K)
    want = oracle.beaver_matmul(X, Y, A, B, C)
    got, direct = launched_direct(lambda: spin.beaver_matmul(dev(X), dev(Y), dev(A), dev(B), dev(C)))
    assert direct and (got.cpu().numpy().view(np.uint64) == want).all()
    Yt, Bt = (dev(t.transpose(0, 1, 3, 2)) for t in (Y, B))
    Z = dev(C)
    _, direct = launched_direct(lambda: spin.beaver_matmul(dev(X), Yt, dev(A), Bt, Z, out=Z, y_transposed=True))
    assert direct and (Z.cpu().numpy().view(np.uint64) == want).all()


@pytest.mark.parametrize("n,batch,M,N,K", SHAPES)
def test_ring32(n, batch, M, N, K):
    rng = np.random.default_rng(M * 1000 + K + 1)
    X = rng.integers(0, 1 << 32, size=(n, batch, M, K), dtype=np.uint64)
    Y = rng.integers(0, 1 << 32, size=(n, batch, K, N), dtype=np.uint64)
    A, B, C = oracle.dealer_matmul(n, batch, M, N, K, seed=K, l=32)
    want = oracle.beaver_matmul(X, Y, A, B, C, l=32)
    ops = [dev(t.astype(np.uint32), np.int32) for t in (X, Y, A, B, C)]
    got, direct = launched_direct(lambda: spin.ring32.beaver_matmul(*ops))
    assert direct and (got.cpu().numpy().view(np.uint32) == want).all()
    spin.ring32.beaver_matmul(*ops, out=ops[4])
    assert torch.equal(ops[4], got)


@pytest.mark.parametrize("n,batch,M,N,K", SHAPES)
def test_ring128(n, batch, M, N, K):
    rng = np.random.default_rng(M * 1000 + K + 2)
    X = rng.integers(0, 1 << 64, size=(n, batch, M, K, 2), dtype=np.uint64)
    Y = rng.integers(0, 1 << 64, size=(n, batch, K, N, 2), dtype=np.uint64)
    A, B, C = r128.dealer_matmul(n, batch, M, N, K, seed=K)
    want = r128.beaver_matmul(X, Y, A, B, C)
    ops = [dev(t) for t in (X, Y, A, B, C)]
    got, direct = launched_direct(lambda: spin.ring128.beaver_matmul(*ops))
    assert direct and (got.cpu().numpy().view(np.uint64) == want).all()
    spin.ring128.beaver_matmul(*ops, out=ops[4])
    assert torch.equal(ops[4], got)


# Wide and batched products whose operands outgrow the caches between two rounds: there the one launch reads them again for every
# tile, and was 1.3 to 2.8 times slower than the digit kernels that have to be chosen.
@pytest.mark.parametrize("bits,n,batch,M,N,K", [(32, 5, 61, 6, 943, 228), (32, 3, 26, 34, 942, 55), (32, 3, 16, 43, 972, 62), (32, 4, 2, 11, 2004, 304),
                                                (64, 7, 19, 13, 476, 43), (64, 1, 1, 704, 847, 20), (64, 3, 11, 30, 802, 59),
                                                (128, 1, 35, 37, 1717, 19), (128, 4, 28, 16, 178, 35), (128, 1, 1, 561, 1841, 17)])
def test_left_to_the_digit_kernels(bits, n, batch, M, N, K):
    matmul = {32: spin.ring32.beaver_matmul, 64: spin.beaver_matmul, 128: spin.ring128.beaver_matmul}[bits]
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 1000 + K)
    dtype, words = (torch.int32, ()) if bits == 32 else (torch.int64, (2,) if bits == 128 else ())
    w = 32 if bits == 32 else 64
    ops = [torch.empty((n, batch) + s + words, dtype=dtype, device="cuda").random_(-2 ** (w - 1), 2 ** (w - 1) - 1, generator=g)
           for s in ((M, K), (K, N), (M, K), (K, N), (M, N))]
    got, direct = launched_direct(lambda: matmul(*ops))
    assert not direct and torch.equal(got, matmul(*ops, path=spin.VALU))
