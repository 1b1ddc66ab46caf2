"""Products that the library takes by the tile kernel's smaller shapes (64 x 64 over Z_2^64; 64 x 128 and 64 x 64 over Z_2^32), at the edges of their tiles
and where several workgroups share one, an even and an odd number of k-tiles, C in place.  Against the vector-ALU path; exact ring words.
The shape is the library's own answer, and shows in the workspace: the right fragments end behind whole tiles of both sides.  (Every shape
and number of parts by name: test_gpu_named_kernels.py.)"""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu

# n, batch, M, N, K; n > 3 over Z_2^64, so that no product is one of the row kernel
SHAPES64 = [(4, 1, 64, 64, 1500), (4, 1, 65, 64, 700), (5, 1, 63, 65, 1000), (4, 3, 129, 128, 96), (5, 1, 128, 129, 161), (4, 16, 192, 65, 64),
            (6, 1, 250, 301, 785), (8, 1, 1, 640, 2049), (4, 1, 320, 700, 66)]
SHAPES32 = [(2, 1, 64, 128, 2000), (3, 1, 65, 64, 700), (5, 1, 63, 129, 1000), (2, 3, 129, 128, 960), (4, 1, 300, 257, 1610), (1, 8, 192, 65, 640),
            (2, 1, 1024, 1024, 1024), (3, 1, 1, 1280, 4097), (2, 1, 700, 900, 330)]


@pytest.mark.parametrize("bits,n,batch,M,N,K", [(64,) + s for s in SHAPES64] + [(32,) + s for s in SHAPES32])
def test_words(bits, n, batch, M, N, K):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    R, dt, w = (spin, torch.int64, 8) if bits == 64 else (spin.ring32, torch.int32, 4)

    def u(*s):
        return torch.empty(s, dtype=dt, device="cuda").random_(-2 ** (bits - 1), 2 ** (bits - 1) - 1, generator=g)
    ops = u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, N)
    want = R.beaver_matmul(*ops, path=spin.VALU)
    need = R.beaver_matmul_workspace_bytes(n, batch, M, N, K)
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    spin.profile_reset()
    spin.profile_enable(True)
    got = [R.beaver_matmul(*ops, workspace=ws) for _ in range(3)]                        # whatever the order of arrival
    torch.cuda.synchronize()
    spin.profile_enable(False)
    count = {k: spin.profile_read(k)[1] for k in ("gemm_limb", "gemm_direct", "gemm_residue")}
    spin.profile_reset()
    assert count == {"gemm_limb": 3, "gemm_direct": 0, "gemm_residue": 0}, "not a product of the tile kernel"
    assert all(torch.equal(z, want) for z in got)
    name, _ = spin.matmul_way(n, batch, M, N, K, bits=bits)
    assert name in ("half", "quarter")
    rows, columns = (64, 128) if (bits, name) == (32, "half") else (64, 64)
    end = (n + 1) * batch * (-(-M // rows) * rows + -(-N // columns) * columns) // 32 * -(-K // 32) * 1024 * w
    assert end - 64 < int((ws != 0x5A).nonzero()[-1]) + 1 <= end
    R.beaver_matmul(*ops, out=ops[4], workspace=ws)
    assert torch.equal(ops[4], want)
