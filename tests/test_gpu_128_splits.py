"""Products over Z_2^128 whose output tiles are shared by several workgroups (128-bit additions made of two 64-bit atomic ones), against
the vector-ALU path: two to sixteen parts, ragged tiles and parts, in place, an inner dimension of several launches, and C and operands
whose sums carry out of the low word every time or never."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu
R = spin.ring128


@pytest.mark.parametrize("n,batch,M,N,K", [(1, 1, 32, 64, 608), (5, 5, 32, 32, 1280), (3, 2, 33, 31, 450), (2, 1, 130, 100, 331), (7, 1, 54, 331, 603), (1, 1, 3, 1, 20000),
                                           (4, 1, 64, 64, 5440), (4, 1, 65, 63, 5473), (3, 1, 384, 160, 1024), (8, 1, 17, 19, 297)])
@pytest.mark.parametrize("values", ["uniform", "high", "low"])
def test_words(n, batch, M, N, K, values):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)

    def u(*s):
        t = torch.empty(s + (2,), dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)
        if values == "high":
            t[..., 0] = -1                               # every addition to a low word carries, or nearly
        elif values == "low":
            t[..., 0] &= 1
        return t
    X, Y, A, B, C = u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, N)
    want = R.beaver_matmul(X, Y, A, B, C, path=spin.VALU)
    # in the workspace that the digit kernels need: a residue product does not fit it in one block
    ws = torch.empty(R.beaver_matmul_workspace_bytes(n, batch, M, N, K), dtype=torch.uint8, device="cuda")
    spin.profile_reset()
    spin.profile_enable(True)
    got = [R.beaver_matmul(X, Y, A, B, C, workspace=ws) for _ in range(3)]               # whatever the order of arrival
    got.append(R.beaver_matmul(X, Y, A, B, C, out=C, workspace=ws))
    torch.cuda.synchronize()
    spin.profile_enable(False)
    count = {k: spin.profile_read(k)[1] for k in ("gemm_limb", "gemm_direct", "gemm_residue")}
    spin.profile_reset()
    assert count == {"gemm_limb": 4 * ((K + 5439) // 5440), "gemm_direct": 0, "gemm_residue": 0}, "goes to another kernel now"
    assert all(torch.equal(z, want) for z in got)
