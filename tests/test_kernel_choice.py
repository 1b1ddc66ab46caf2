"""The choice between residue and digit GEMMs shows in the preferred workspace: above the required one only where the residue GEMM is
taken.  Products that it was slower on (measured, us by digits against residues, behind each) stay with the digit kernels; clear
ones go to it.  The queries touch no GPU; without one the library reckons with 256 CUs."""
import pytest

from paper_2402_02320_amd import spin

DIGITS = [(128, 3, 1, 320, 128, 96),        # 34 : 63
          (128, 4, 1, 77, 245, 99),         # 43 : 73
          (128, 2, 1, 736, 128, 96),        # 40 : 57
          (128, 4, 1, 192, 128, 160),       # 46 : 69
          (128, 6, 1, 64, 224, 288),        # 44 : 94
          (128, 6, 1, 64, 608, 1120),       # 113 : 250
          (128, 5, 2, 63, 52, 1950),        # 61 : 296, tiles shared by several workgroups from here on
          (128, 2, 1, 48, 48, 2000),        # 44 : 83
          (128, 2, 1, 49, 49, 2000),        # 45 : 87
          (128, 3, 1, 64, 64, 699),         # 34 : 71
          (128, 3, 1, 64, 64, 700),         # 34 : 70
          (128, 8, 1, 49, 50, 5835),        # 174 : 641
          (128, 1, 1, 300, 300, 5440),      # 158 : 268, one launch of the digit GEMM
          (128, 1, 1, 300, 300, 5441),      # 177 : 265, two
          (128, 5, 1, 163, 161, 1460),      # 93 : 138
          (128, 3, 1, 480, 128, 3392),      # 221 : 248
          (64, 1, 1, 1504, 800, 512),       # 52 : 62
          (64, 4, 1, 466, 807, 2203),       # 242 : 271
          (64, 5, 1, 130, 1643, 716),       # 140 : 152
          (64, 3, 1, 256, 2976, 608)]       # 140 : 151
RESIDUES = [(128, 2, 1, 2048, 2048, 2048), (128, 3, 1, 1024, 512, 1024), (128, 4, 1, 512, 640, 2000), (128, 2, 1, 160, 2336, 1696),
            (128, 2, 1, 512, 512, 5440), (128, 2, 1, 512, 512, 5441),     # 679 : 555, 700 : 562
            (64, 2, 1, 2048, 2048, 2048), (64, 5, 1, 4096, 4096, 4096)]


@pytest.mark.parametrize("bits,n,batch,M,N,K,residue", [d + (False,) for d in DIGITS] + [d + (True,) for d in RESIDUES])
def test_residue_or_digits(bits, n, batch, M, N, K, residue):
    pre = "spin" if bits == 64 else "spin128"
    need, preferred = (getattr(spin.lib(), pre + "_beaver_matmul_" + q) for q in ("workspace_bytes", "preferred_workspace_bytes"))
    args = (n, batch, M, N, K, spin.LIMB_MFMA)
    assert (preferred(*args) > need(*args)) is residue


def test_no_workspace_of_gigabytes_for_a_hundredth():
    # 3.5 GB in two blocks are estimated (and measured) no slower than 5.1 GB in one
    q = spin.beaver_matmul_preferred_workspace_bytes
    assert spin.beaver_matmul_workspace_bytes(5, 1, 4096, 4096, 4096) < q(5, 1, 4096, 4096, 4096) < 4e9
    assert spin.beaver_matmul_workspace_bytes(3, 1, 4096, 4096, 2048) < q(3, 1, 4096, 4096, 2048) < 1e9
    assert spin.ring128.beaver_matmul_preferred_workspace_bytes(2, 1, 2048, 2048, 2048) > 1e9     # 4 % faster than in 0.75 GB


@pytest.mark.parametrize("n,batch,M,together", [(1, 15, 1 << 24, True), (1, 16, 1 << 24, False), (1, 16, (1 << 24) - 32, True), (1, 16, (1 << 24) - 31, False),
                                                (3, 17, 1 << 24, False)])
def test_a_grouped_call_of_more_threads_than_a_grid_holds_is_taken_apart(n, batch, M, together):
    # one workgroup of 512 threads to 32 rows: 2^23 of them are a grid of 2^32 threads, which HIP refuses
    assert (spin.matmul_grouped_way(n, [(batch, M, 1, 1)]) == "rows") is together
    assert (spin.matmul_grouped_way(n, [(batch, M, 1, 1), (1, 8, 8, 8)]) == "rows") is together
