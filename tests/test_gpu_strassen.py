"""Large products over Z_2^32 by two levels of Strassen's recursion: the words of the digit kernels alone (which the same call takes in
the workspace it needs), where all sides are ragged, in place, over batch entries; and where the workspace is too small by a byte."""
import pytest
import torch

from paper_2402_02320_amd import spin

R = spin.ring32
# rows of 16 bytes and not, on either side; one party; one and several batch entries and parties; last blocks that are full and as empty
# as blocks in multiples of 128 leave them (1025 of 1536 rows, 1537 of 2048)
SHAPES = [(2, 1, 7159, 5629, 8785), (1, 1, 8192, 8190, 8188), (1, 2, 8189, 8192, 8064), (3, 1, 5059, 7112, 7399), (2, 2, 6144, 6144, 6144),
          (2, 1, 5633, 6144, 8192), (1, 1, 7681, 8192, 8191)]
# measured, us by the digit kernels and by the recursion, in the workspace that each needs
FASTER = [(2, 1, 6592, 10016, 7328), (4, 1, 3488, 5632, 7424), (3, 1, 4032, 7680, 7680)]           # 15907 : 14081, 9582 : 8434, 11791 : 10455
SLOWER = [(2, 1, 4096, 4096, 2048), (4, 1, 9376, 3776, 4192)]                                      # the second 9518 : 9564


def test_only_large_products_prefer_more_workspace():
    for dims in SHAPES + FASTER:
        assert R.beaver_matmul_preferred_workspace_bytes(*dims) > 2 * R.beaver_matmul_workspace_bytes(*dims)
    for dims in SLOWER + [(2, 1, 8192, 64, 8192), (5, 1, 300, 300, 300), (2, 64, 512, 512, 512)]:
        assert R.beaver_matmul_preferred_workspace_bytes(*dims) == R.beaver_matmul_workspace_bytes(*dims)
    assert R.beaver_matmul_preferred_workspace_bytes(0, 1, 8192, 8192, 8192) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dims", SHAPES)
def test_words_of_the_digit_kernels(dims):
    n, batch, M, N, K = dims
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)

    def u(*s):
        return torch.empty(s, dtype=torch.int32, device="cuda").random_(-2 ** 31, 2 ** 31 - 1, generator=g)
    X, Y, A, B, C = u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, N)
    most = torch.empty(R.beaver_matmul_preferred_workspace_bytes(*dims), dtype=torch.uint8, device="cuda")

    def combines(workspace, out):
        spin.profile_reset()
        spin.profile_enable(True)
        Z = R.beaver_matmul(X, Y, A, B, C, out=out, workspace=workspace)
        torch.cuda.synchronize()
        spin.profile_enable(False)
        count = spin.profile_read("combine")[1]
        spin.profile_reset()
        return Z, count
    want, count = combines(most[:most.numel() - 256], None)
    assert count == 0
    got, count = combines(most, None)
    assert count == 1 and torch.equal(got, want)
    combines(most, C)                                    # in place
    assert torch.equal(C, want)
