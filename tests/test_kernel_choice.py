"""The choice between residue and digit GEMMs shows in the preferred workspace: above the required one only where the residue GEMM is
taken.  Products that it was slower on (measured, us by digits against residues, behind each) stay with the digit kernels; clear
ones go to it.  The queries touch no GPU; without one the library reckons with 256 CUs."""
import pytest

from paper_2402_02320_amd import spin

DIGITS = [(128, 3, 1, 320, 128, 96),        # 34 : 63
          (128, 4, 1, 77, 245, 99),         # 43 : 73
          (128, 2, 1, 736, 128, 96),        # 40 : 57
          (128, 4, 1, 192, 128, 160),       # 46 : 69
          (128, 6, 1, 64, 224, 288),        # 76 : 93
          (128, 6, 1, 64, 608, 1120),       # 235 : 246
          (64, 1, 1, 1504, 800, 512),       # 52 : 62
          (64, 4, 1, 466, 807, 2203),       # 242 : 271
          (64, 5, 1, 130, 1643, 716),       # 140 : 152
          (64, 3, 1, 256, 2976, 608)]       # 140 : 151
RESIDUES = [(128, 2, 1, 2048, 2048, 2048), (128, 3, 1, 480, 128, 3392), (128, 4, 1, 103, 2467, 1327), (128, 2, 1, 160, 2336, 1696),
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
