"""Every kind of plan that the residue GEMM computes a product by, chosen through the workspace it is given: groups of one party,
blocks of rows and of columns of panels, even and uneven, operands that stay converted from block to block, several chunks of the
inner dimension, batches, and items shared in parts, with wide and narrow tiles.  `blocks` is what the plan comes to for this
workspace, and the number of launches that the library reports; a case that fails there has to be chosen anew.  Over Z_2^64 the residue
GEMM is asked for by name (some of these products are faster by tiles).  Against the vector-ALU path, in a workspace that starts out dirty; random operands, exact words."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu

# n, batch, M, N, K, transposed, workspace, blocks
CASES64 = [(2, 1, 389, 2224, 1193, True, 227377151, 2),       # one party at a time, transposed, odd K, wide tiles in two parts
           (2, 2, 1221, 1234, 804, True, 173998079, 4),       # one party at a time, two batch entries
           (2, 1, 389, 1613, 5796, True, 399310847, 4),       # one party at a time, two chunks of K
           (2, 1, 1263, 2435, 823, False, 173998079, 4),      # one party at a time, two blocks of columns
           (3, 1, 660, 983, 1160, True, 199360511, 2),        # left operands kept over two blocks of columns, transposed
           (3, 1, 396, 1423, 5749, False, 467140607, 4),      # the same over two chunks, items in three parts
           (3, 2, 401, 2281, 1106, False, 297271295, 4),      # right operands kept over two blocks of rows, two batch entries
           (3, 1, 1431, 1513, 1105, False, 169869311, 4),     # two blocks of rows and two of columns
           (2, 1, 398, 2251, 1569, True, 192348159, 2),       # nine panels of columns in blocks of five and four, in parts
           (2, 1, 1939, 1115, 1537, False, 238878719, 3),     # eight panels of rows in blocks of three, narrow tiles
           (3, 1, 1169, 540, 987, True, 206372864, 1),        # narrow tiles in parts
           (2, 1, 1206, 856, 970, False, 174587903, 2)]       # the same, one party at a time
CASES128 = [(2, 2, 459, 533, 1009, 113246208, 4),             # one party at a time, two batch entries
            (2, 1, 217, 875, 4370, 242417664, 4),             # one party at a time, two chunks
            (2, 1, 386, 1438, 945, 106522214, 4),             # one party at a time, two blocks of columns
            (3, 1, 195, 912, 3790, 298070835, 4),             # left operands kept over two blocks of columns, two chunks
            (3, 2, 1268, 655, 525, 220882534, 4),             # right operands kept over uneven blocks of rows, two batch entries
            (3, 1, 769, 909, 885, 169869311, 4),              # two blocks of rows and two of columns
            (5, 1, 708, 551, 748, 334784102, 2),              # three panels of rows in blocks of two and one, narrow tiles
            (5, 1, 1037, 338, 5143, 849720115, 4),            # five panels in blocks of three and two, items in parts, two chunks
            (2, 1, 961, 259, 4312, 401866752, 2),             # narrow tiles in parts, two chunks
            (3, 1, 197, 666, 4398, 360448000, 2),             # wide tiles in parts, two chunks
            (2, 1, 2048, 2048, 2048, 402653184, 8)]           # the workspace that is needed: wide tiles in four parts


def run(bits, n, batch, M, N, K, transposed, size, blocks):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    words, y = (2,) if bits == 128 else (), (N, K) if transposed else (K, N)
    X, Y, A, B, C = (torch.empty((n, batch) + s + words, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)
                     for s in ((M, K), y, (M, K), y, (M, N)))
    matmul = spin.beaver_matmul if bits == 64 else spin.ring128.beaver_matmul
    kw = {"y_transposed": True} if transposed else {}
    want = matmul(X, Y, A, B, C, path=spin.VALU, **kw)
    if bits == 64:
        matmul = lambda *ops, **k: spin.beaver_matmul_by("residues", 1, *ops, **k)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda").random_(0, 256, generator=g)
    spin.profile_reset()
    spin.profile_enable(True)
    got = matmul(X, Y, A, B, C, workspace=ws, **kw)
    torch.cuda.synchronize()
    spin.profile_enable(False)
    count = {k: spin.profile_read(k)[1] for k in ("gemm_residue", "combine", "gemm_limb", "gemm_direct")}
    spin.profile_reset()
    assert count == {"gemm_residue": blocks, "combine": blocks, "gemm_limb": 0, "gemm_direct": 0}
    assert torch.equal(got, want)
    matmul(X, Y, A, B, C, out=C, workspace=ws, **kw)             # in place, over what the first call left behind
    assert torch.equal(C, want)


@pytest.mark.parametrize("n,batch,M,N,K,transposed,size,blocks", CASES64)
def test_ring64(n, batch, M, N, K, transposed, size, blocks):
    run(64, n, batch, M, N, K, transposed, size, blocks)


@pytest.mark.parametrize("n,batch,M,N,K,size,blocks", CASES128)
def test_ring128(n, batch, M, N, K, size, blocks):
    run(128, n, batch, M, N, K, False, size, blocks)
