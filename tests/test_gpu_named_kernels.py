"""Every digit kernel by its name: each tile shape over Z_2^64 and Z_2^32 at the edges of its tiles, whole and with several workgroups to a tile, the
row kernel at the largest sums that its accumulators may hold, and a grouped call by each of its kernels.  Against the vector-ALU path or a closed
form; exact ring words.  That a tile product came in tiles of the named shape shows in the workspace: the right fragments end behind
whole tiles of both sides."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu

TILES = {(64, "full"): (128, 64), (64, "half"): (64, 64), (32, "full"): (128, 128), (32, "half"): (64, 128), (32, "quarter"): (64, 64)}


def uniform(seed, bits=64):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dtype = torch.int64 if bits == 64 else torch.int32
    return lambda *s: torch.empty(s, dtype=dtype, device="cuda").random_(-2 ** (bits - 1), 2 ** (bits - 1) - 1, generator=g)


# n, batch, rows beyond whole tiles, tiles of rows, columns beyond, tiles of columns, K, parts.  k-tiles and parts: 16 of one k-tile (two k-steps) each, 3 of 6, 6
# and 5, 11 of 3; one, two and three k-tiles alone; a last k-tile of 1, 31 and 32.
CASES = [(4, 1, 0, 1, 0, 1, 512, 1), (4, 1, 0, 1, 0, 1, 512, 16), (5, 2, 1, 1, -1, 2, 513, 3), (2, 1, -1, 2, 1, 1, 1055, 11), (1, 3, -63, 1, -63, 1, 32, 1),
         (3, 1, 1, 2, 1, 2, 33, 2), (8, 1, 0, 2, 0, 1, 95, 3), (3, 2, -1, 1, -1, 1, 96, 1), (6, 1, 0, 1, 1, 1, 640, 2)]


@pytest.mark.parametrize("bits,name", sorted(TILES))
@pytest.mark.parametrize("n,batch,dm,tm,dn,tn,K,parts", CASES)
def test_tiles(bits, name, n, batch, dm, tm, dn, tn, K, parts):
    rows, columns = TILES[bits, name]
    M, N = rows * tm + dm, columns * tn + dn
    u, R = uniform(M + N + K, bits), spin if bits == 64 else spin.ring32
    ops = u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, K), u(n, batch, K, N), u(n, batch, M, N)
    want = R.beaver_matmul(*ops, path=spin.VALU)
    ws = torch.full((R.beaver_matmul_workspace_bytes(n, batch, M, N, K),), 0x5A, dtype=torch.uint8, device="cuda")
    for _ in range(3):                                                                   # whatever the order of arrival
        assert torch.equal(spin.beaver_matmul_by(name, parts, *ops, workspace=ws), want)
    end = (n + 1) * batch * (-(-M // rows) * rows + -(-N // columns) * columns) // 32 * -(-K // 32) * 1024 * (bits // 8)
    assert end - 64 < int((ws != 0x5A).nonzero()[-1]) + 1 <= end
    if bits == 64:
        Yt, Bt = (t.transpose(2, 3).contiguous() for t in (ops[1], ops[3]))
        assert torch.equal(spin.beaver_matmul_by(name, parts, ops[0], Yt, ops[2], Bt, ops[4], y_transposed=True), want)
    spin.beaver_matmul_by(name, parts, *ops, out=ops[4])
    assert torch.equal(ops[4], want)


@pytest.mark.parametrize("name", ["full", "half"])
@pytest.mark.parametrize("K,parts", [(512 * 32 + 40, 1), (511 * 32 + 1, 7), (600 * 32, 16)])
def test_an_inner_dimension_of_two_launches(name, K, parts):
    u = uniform(K)
    ops = u(2, 1, 5, K), u(2, 1, K, 70), u(2, 1, 5, K), u(2, 1, K, 70), u(2, 1, 5, 70)
    want = spin.beaver_matmul(*ops, path=spin.VALU)
    assert torch.equal(spin.beaver_matmul_by(name, parts, *ops), want)
    spin.beaver_matmul_by(name, parts, *ops, out=ops[4])
    assert torch.equal(ops[4], want)


@pytest.mark.parametrize("name,parts", [("rows", 1), ("full", 1), ("half", 1), ("half", 7)])
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("M,N", [(33, 64), (64, 33), (1, 65)])
def test_largest_sums(name, parts, n, M, N):
    # all digits of E, F, A_p and B_p -128 over the longest inner dimension that is accumulated at once: 511 k-tiles
    K, w, m = 511 * 32, 0x7F7F7F7F7F7F7F80, 1 << 64
    worst = torch.tensor(w, dtype=torch.int64, device="cuda")
    X, Y = worst.expand(n, 1, M, K).contiguous(), worst.expand(n, 1, K, N).contiguous()
    A, B = X.clone(), Y.clone()
    A[0], B[0] = 0, 0
    got = spin.beaver_matmul_by(name, parts, X, Y, A, B, torch.zeros(n, 1, M, N, dtype=torch.int64, device="cuda"))
    for i in range(n):                                   # E = F = w; Z_0 = E (B_0 + F) + A_0 F, Z_i = E B_i + A_i F
        v = (1 if i == 0 else 2) * K * w * w % m
        assert bool((got[i] == (v - m if v >> 63 else v)).all())


SHAPES = [(2, 196, 96, 64, True), (3, 49, 32, 49, False), (1, 33, 64, 130, False), (2, 70, 65, 33, True), (1, 1, 1, 2, False), (1, 5, 7, 1, True)]


@pytest.mark.parametrize("n,name", [(n, name) for n in (1, 2, 3, 4) for name in ("rows", "full", "half") if n < 4 or name != "rows"])
@pytest.mark.parametrize("count", [1, 6, 36])                                            # of 36 the sides take two launches or three
def test_grouped(n, name, count):
    u, groups = uniform(n * 100 + count), []
    for batch, M, N, K, transposed in (SHAPES * 6)[:count]:
        y = (N, K) if transposed else (K, N)
        groups.append(dict(X=u(n, batch, M, K), Y=u(n, batch, *y), A=u(n, batch, M, K), B=u(n, batch, *y), C=u(n, batch, M, N), y_transposed=transposed))
    want = spin.beaver_matmul_grouped(groups, path=spin.VALU)
    for _ in range(2):
        assert all(torch.equal(a, b) for a, b in zip(spin.beaver_matmul_grouped_by(name, groups), want))


@pytest.mark.parametrize("bits", [64, 32])
def test_direct(bits):
    u, R = uniform(5, bits), spin if bits == 64 else spin.ring32
    ops = u(3, 2, 65, 300), u(3, 2, 300, 130), u(3, 2, 65, 300), u(3, 2, 300, 130), u(3, 2, 65, 130)
    assert torch.equal(spin.beaver_matmul_by("direct", 1, *ops), R.beaver_matmul(*ops, path=spin.VALU))


def test_residues():
    u = uniform(1)
    ops = u(2, 1, 300, 700), u(2, 1, 700, 270), u(2, 1, 300, 700), u(2, 1, 700, 270), u(2, 1, 300, 270)
    ws = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    spin.profile_reset()
    spin.profile_enable(True)
    got = spin.beaver_matmul_by("residues", 1, *ops, workspace=ws)
    torch.cuda.synchronize()
    spin.profile_enable(False)
    launches = spin.profile_read("gemm_residue")[1]
    spin.profile_reset()
    assert launches == 1 and torch.equal(got, spin.beaver_matmul(*ops, path=spin.VALU))
