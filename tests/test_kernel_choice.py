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


def test_a_grouped_call_of_more_threads_than_a_grid_holds_is_taken_apart():
    # 2^32 threads and more, which HIP refuses: 2^23 row blocks of 512 threads, 2^24 tiles of 256
    SEPARATE, ERANGE, M = "separate", 2, 1 << 24
    assert spin.matmul_grouped_way(1, [(64, M, 1, 1)]) == spin.matmul_grouped_way(1, [(63, M, 1, 1), (1, M, 1, 1)]) == SEPARATE
    assert spin.matmul_grouped_way(1, [(63, M, 1, 1)]) != SEPARATE
    for n, shapes in ((1, [(16, M)]), (1, [(16, M - 31)]), (1, [(15, M), (1, M)]), (3, [(17, M)])):
        desc = (spin._MatmulGroup * len(shapes))()
        for d, (batch, rows) in zip(desc, shapes):
            d.batch, d.M, d.N, d.K = batch, rows, 1, 1
            d.X = d.Y = d.A = d.B = d.C = d.Z = 0x10000      # never touched: refused before anything is launched
        assert spin.lib().spin_matmul_grouped_by(spin._MatmulWay(spin.WAYS["rows"], 1), n, len(shapes), desc, 0x10000, 1 << 50, None) == ERANGE


# us by the way that is taken, and by the one behind it
WAYS = [((3, 1, 256, 190, 130), "tiles"),           # 15.4, 25.9 by rows
        ((3, 7, 20, 190, 130), "tiles"),            # 18.8, 27.5 by rows
        ((3, 3, 129, 129, 66), "tiles"),            # 15.7, 21.8 by rows
        ((3, 1, 512, 128, 66), "tiles"),            # 15.2, 20.6 by rows
        ((3, 1, 472, 108, 157), "tiles"),           # 16.7, 27.2 by rows
        ((3, 1, 5006, 69, 113), "tiles"),           # 28.7, 37.7 by rows
        ((3, 1, 2233, 2432, 131), "tiles"),         # 196, 252 by rows: many column tiles, each of which reads the rows again
        ((2, 14, 704, 960, 736), "tiles"),          # 939, 1145 by rows
        ((3, 1, 7840, 2112, 160), "tiles"),         # 558, 718 by rows
        ((3, 64, 128, 128, 64), "rows"),            # 32.5
        ((3, 61, 3851, 83, 33), "rows"),            # 536, 624 by half tiles
        ((3, 1, 131072, 64, 576), "rows"),          # 1140
        ((2, 1, 4200, 64, 16352), "rows"),
        ((2, 1, 1024, 1024, 1024), "full")]         # 130, 135 by half tiles


@pytest.mark.parametrize("dims,name", WAYS)
def test_rows_or_tiles(dims, name):
    assert spin.matmul_way(*dims)[0] in (("full", "half") if name == "tiles" else (name,))


@pytest.mark.parametrize("dims", [(2, 1, 389, 2224, 1193), (2, 1, 398, 2251, 1569), (3, 1, 1169, 540, 987)])
def test_tiles_in_parts_or_residues(dims):
    # us by tiles, by residues in one block or two: 160 : 207, 212 : 244, 152 : 163
    assert spin.beaver_matmul_preferred_workspace_bytes(*dims) == spin.beaver_matmul_workspace_bytes(*dims)


@pytest.mark.parametrize("n,scale,name", [(3, 1, "half"), (3, 2, "half"), (3, 3, "rows"), (3, 8, "rows"), (2, 1, "rows"), (2, 8, "rows")])
def test_grouped_rows_or_tiles(n, scale, name):
    # six attention products of three stages, by rows and half tiles: 33.6 : 28.4, 44.7 : 38.2, 45.9 : 48.9, 110 : 127; two parties 26.3 : 28.6, 74 : 86
    shapes = [(4, 196, 196, 64, True), (4, 196, 64, 196), (8, 49, 49, 32, True), (8, 49, 32, 49), (12, 16, 16, 32, True), (12, 16, 32, 16)]
    assert spin.matmul_grouped_way(n, [(scale * s[0],) + s[1:] for s in shapes]) == name
    if n == 3:
        assert spin.matmul_grouped_way(3, [(1, 1024, 1024, 160)] * 2) == "half"              # 52 : 62 us; five k-tiles
