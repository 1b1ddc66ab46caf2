"""The packs of the digit kernels as one launch or as one a side, with the copy of C in the pack or by itself: products on both
sides of every line that chooses between them, out of place and in place, against the vector-ALU path.  Exact ring words."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu


def uniform(g, *shape, dtype=torch.int64):
    w = 32 if dtype == torch.int32 else 64
    return torch.empty(shape, dtype=dtype, device="cuda").random_(-2 ** (w - 1), 2 ** (w - 1) - 1, generator=g)


# over Z_2^128 a row block of 64 and 32 k make one workgroup of the left pack: 512, 513 (beyond one wave per SIMD of 256 CUs) of them;
# then one side, the other, both past the caches (non-temporal)
@pytest.mark.parametrize("n,batch,M,N,K", [(2, 1, 2048, 20, 512), (2, 1, 2049, 20, 512), (2, 9, 192, 33, 609), (1, 1, 2049, 20, 512),
                                           (3, 1, 2100, 40, 512), (2, 1, 8200, 1, 512), (2, 1, 1, 8200, 512), (8, 2, 1000, 70, 300)])
def test_ring128(n, batch, M, N, K):
    run(spin.ring128.beaver_matmul, n, batch, M, N, K, (2,), torch.int64)


# 23 MB of C, a little less and a little more, where several workgroups share a tile, 8 MB where one side streams; one side, both sides past the caches
@pytest.mark.parametrize("n,batch,M,N,K", [(5, 1, 640, 640, 1024), (5, 1, 1024, 1024, 1024), (7, 1, 512, 841, 2000), (7, 1, 512, 842, 2000),
                                           (4, 1, 64, 4096, 1100), (4, 1, 65, 4096, 1100), (4, 1, 4099, 60, 1100), (5, 1, 1700, 1300, 1301), (7, 3, 100, 120, 1001)])
def test_ring64(n, batch, M, N, K):
    for transposed in (False, True):
        run(spin.beaver_matmul, n, batch, M, N, K, (), torch.int64, transposed)


# whole and ragged tiles, left (right) operands past the caches, rows of 16 and of 8 bytes, for the party counts whose shares take the most registers
@pytest.mark.parametrize("n,batch,M,N,K", [(8, 1, 1208, 320, 1056), (8, 1, 1205, 70, 1067), (7, 1, 70, 1210, 1057), (6, 2, 133, 165, 297), (8, 2, 131, 163, 295)])
def test_many_parties(n, batch, M, N, K):
    for transposed in (False, True):
        run(spin.beaver_matmul, n, batch, M, N, K, (), torch.int64, transposed)


@pytest.mark.parametrize("n,batch,M,N,K", [(5, 1, 16384, 128, 576), (7, 1, 32, 2048, 2048), (4, 1, 300, 500, 3001), (3, 2, 2000, 1000, 96)])
def test_ring32(n, batch, M, N, K):
    run(spin.ring32.beaver_matmul, n, batch, M, N, K, (), torch.int32)


def run(matmul, n, batch, M, N, K, words, dtype, transposed=False):
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 3 + K)
    y = (N, K) if transposed else (K, N)
    X, Y, A, B, C = (uniform(g, n, batch, *s, *words, dtype=dtype) for s in ((M, K), y, (M, K), y, (M, N)))
    kw = dict(y_transposed=True) if transposed else {}
    # the workspace that the digit kernels need and no more: a residue product of these sizes does not fit it
    L, pre = spin.lib(), {torch.int32: "spin32", torch.int64: "spin128" if words else "spin"}[dtype]
    ws = torch.empty(getattr(L, pre + "_beaver_matmul_workspace_bytes")(n, batch, M, N, K, spin.LIMB_MFMA), dtype=torch.uint8, device="cuda")
    if dtype == torch.int64:
        kw["workspace"] = ws
    want = matmul(X, Y, A, B, C, path=spin.VALU, **({"y_transposed": True} if transposed else {}))
    spin.profile_reset()
    spin.profile_enable(True)
    got = matmul(X, Y, A, B, C, **kw)
    torch.cuda.synchronize()
    spin.profile_enable(False)
    packs = spin.profile_read("pack")[1], spin.profile_read("gemm_limb")[1]
    spin.profile_reset()
    assert packs[0] == 1 and packs[1] >= 1, "not a product of the digit kernels any more"
    assert torch.equal(got, want)
    matmul(X, Y, A, B, C, out=C, **kw)
    assert torch.equal(C, want)
