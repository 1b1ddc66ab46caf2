"""The residue GEMM (large products over Z_2^64 and Z_2^128) against the CPU oracle and the VALU path: partial panels and
k-steps, a second inner-dimension chunk, transposed right operands, some plans of several blocks (the others are in
test_gpu_residue_plans.py), and operands whose digits are all extreme; the same products in place on C in the workspace that
the call needs, where they mostly go to the digit kernels.  Results are ring words, so equality is exact."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from oracle import r128
from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu


def uniform(g, *shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)


def operands(seed, n, batch, M, N, K, transposed=False, words=()):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    y = (N, K) if transposed else (K, N)
    return (uniform(g, n, batch, M, K, *words), uniform(g, n, batch, *y, *words), uniform(g, n, batch, M, K, *words),
            uniform(g, n, batch, *y, *words), uniform(g, n, batch, M, N, *words))


def host(t):
    return np.ascontiguousarray(t.cpu().numpy().view(np.uint64))


def preferred(L, bits, *dims):
    f = L.spin_beaver_matmul_preferred_workspace_bytes if bits == 64 else L.spin128_beaver_matmul_preferred_workspace_bytes
    return int(f(*dims, spin.LIMB_MFMA))


# n, batch, M, N, K, transposed
SHAPES64 = [(5, 1, 1025, 1200, 1001, False),      # odd K (no 16-byte rows), one row beyond four panels
            (8, 1, 769, 1023, 1100, True),        # right operand stored transposed, eight parties
            (2, 1, 1300, 1300, 5633, False),      # one k beyond a launch: two chunks, the second onto Z
            (2, 2, 1500, 1030, 1600, False),      # two batch entries
            (3, 1, 2048, 1024, 1537, True),       # odd K, transposed
            (4, 1, 1024, 1024, 1088, False),      # 4.5 rounds of workgroups: the last items come in two parts
            (2, 1, 1500, 1500, 1400, False)]     # 5.06 rounds: a few items in several parts


@pytest.mark.parametrize("n,batch,M,N,K,transposed", SHAPES64)
def test_ring64(n, batch, M, N, K, transposed):
    dims = (n, batch, M, N, K)
    X, Y, A, B, C = operands(K, n, batch, M, N, K, transposed)
    want = spin.beaver_matmul(X, Y, A, B, C, path=spin.VALU, y_transposed=transposed)
    ample = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    got = spin.beaver_matmul_by("residues", 1, X, Y, A, B, C, workspace=ample, y_transposed=transposed)
    assert torch.equal(got, want)
    assert torch.equal(spin.beaver_matmul(X, Y, A, B, C, y_transposed=transposed), want)         # the way that the library takes
    rows = np.unique(np.array([0, 15, 16, 127, 128, 255, 256, M // 2, M - 2, M - 1], dtype=np.int32) % M)
    Yh, Bh = (host(t.transpose(2, 3) if transposed else t) for t in (Y, B))
    assert (host(got)[:, :, rows] == oracle.beaver_matmul(host(X), Yh, host(A), Bh, host(C), rows=rows)).all()
    # in place on C, twice on one workspace of the size that is needed (block by block, or the digit kernels)
    ws = torch.empty(spin.beaver_matmul_workspace_bytes(*dims), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        Z = C.clone()
        spin.beaver_matmul(X, Y, A, B, Z, out=Z, workspace=ws, y_transposed=transposed)
        assert torch.equal(Z, want)


@pytest.mark.parametrize("n,M,N,K", [(5, 2048, 2048, 2048), (4, 2100, 2000, 4000), (3, 4096, 2048, 2048), (2, 4096, 4096, 4096)])
def test_ring64_block_plans(n, M, N, K):
    # workspaces between what is needed and what is preferred: different groups of parties and panels, the same words
    X, Y, A, B, C = operands(n, n, 1, M, N, K)
    want = spin.beaver_matmul(X, Y, A, B, C, path=spin.VALU)
    need, most = spin.beaver_matmul_workspace_bytes(n, 1, M, N, K), preferred(spin.lib(), 64, n, 1, M, N, K)
    assert most > need
    for size in sorted({need, need + (most - need) // 8, (need + most) // 2, most}):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        assert torch.equal(spin.beaver_matmul(X, Y, A, B, C, workspace=ws), want), size
        del ws


@pytest.mark.parametrize("n,batch,M,N,K", [(3, 1, 512, 512, 700), (2, 1, 769, 400, 701), (1, 1, 510, 760, 3713), (2, 2, 600, 560, 1000),
                                           (2, 1, 600, 390, 1001)])
def test_ring128(n, batch, M, N, K):
    dims = (n, batch, M, N, K)
    X, Y, A, B, C = operands(K, n, batch, M, N, K, words=(2,))
    assert preferred(spin.lib(), 128, *dims) > spin.ring128.beaver_matmul_workspace_bytes(*dims), "not a residue product any more"
    want = spin.ring128.beaver_matmul(X, Y, A, B, C, path=spin.VALU)
    got = spin.ring128.beaver_matmul(X, Y, A, B, C)
    assert torch.equal(got, want)
    if M * N * K < 2e8:
        assert (host(got) == r128.beaver_matmul(host(X), host(Y), host(A), host(B), host(C))).all()
    Z = C.clone()
    ws = torch.empty(spin.ring128.beaver_matmul_workspace_bytes(*dims), dtype=torch.uint8, device="cuda")
    spin.ring128.beaver_matmul(X, Y, A, B, Z, out=Z, workspace=ws)
    assert torch.equal(Z, want)


@pytest.mark.parametrize("bits,M,N,K", [(64, 1280, 1280, 5632), (128, 512, 512, 3712)])
@pytest.mark.parametrize("left,right", [(0x80, 0x80), (0x7F, 0x7F), (0x80, 0x7F)])
def test_extreme_digits(bits, M, N, K, left, right):
    # digits at the ends of their range over the longest inner dimension of one launch; in the second product those of
    # all four operands: the largest sums the reconstruction can meet
    def fill(byte, rows, cols):
        w = int.from_bytes(bytes([byte] * 8), "little", signed=True)
        return torch.full((1, 1, rows, cols) + ((2,) if bits == 128 else ()), w, dtype=torch.int64, device="cuda")
    mod = spin.ring128 if bits == 128 else spin
    dims = (1, 1, M, N, K)
    assert preferred(spin.lib(), bits, *dims) > mod.beaver_matmul_workspace_bytes(*dims), "not a residue product any more"
    A, B = fill(left, M, K), fill(right, K, N)
    a, b = (int.from_bytes(bytes([v] * (bits // 8)), "little") for v in (left, right))
    X, Y = fill(left, M, K), fill(right, K, N)                # E = X - A = left, F = Y - B = right: X = 2 left, Y = 2 right
    for t, v in ((X, 2 * a), (Y, 2 * b)):
        for w in range(bits // 64):
            word = (v >> (64 * w)) & (2 ** 64 - 1)
            (t[..., w] if bits == 128 else t).fill_(word - 2 ** 64 if word >> 63 else word)
    C = torch.zeros_like(fill(0, M, N))
    # Z = E.(B + F) + A.F
    want = (K * (a * (2 * b) + a * b)) % (1 << bits)
    got = mod.beaver_matmul(X, Y, A, B, C)
    for w in range(bits // 64):
        word = (want >> (64 * w)) & (2 ** 64 - 1)
        assert bool(((got[..., w] if bits == 128 else got) == (word - 2 ** 64 if word >> 63 else word)).all())
    B0 = torch.zeros_like(B)
    got = mod.beaver_matmul(X, B, A, B0, C)                   # F = B, B' = B: all four operands extreme
    want = (2 * K * a * b) % (1 << bits)
    for w in range(bits // 64):
        word = (want >> (64 * w)) & (2 ** 64 - 1)
        assert bool(((got[..., w] if bits == 128 else got) == (word - 2 ** 64 if word >> 63 else word)).all())


def test_graph_replays():
    n, M, N, K = 3, 1536, 1536, 1536
    X, Y, A, B, C = operands(9, n, 1, M, N, K)
    ws = torch.empty(preferred(spin.lib(), 64, n, 1, M, N, K), dtype=torch.uint8, device="cuda")
    assert ws.numel() > spin.beaver_matmul_workspace_bytes(n, 1, M, N, K)
    Z = torch.empty_like(C)
    spin.beaver_matmul(X, Y, A, B, C, out=Z, workspace=ws)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            spin.beaver_matmul(X, Y, A, B, C, out=Z, workspace=ws)
    torch.cuda.synchronize()
    for seed in range(3):
        for t, u in zip((X, Y, A, B, C), operands(20 + seed, n, 1, M, N, K)):
            t.copy_(u)
        want = spin.beaver_matmul(X, Y, A, B, C, path=spin.VALU)
        Z.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Z, want), seed


def test_preferred_workspace_query():
    L = spin.lib()
    q, p = L.spin_beaver_matmul_workspace_bytes, L.spin_beaver_matmul_preferred_workspace_bytes
    assert p(0, 1, 4, 4, 4, 0) == 0 and p(2, 1, 4, 4, 4, 5) == 0
    for dims in ((3, 1, 64, 64, 64), (2, 3, 100, 70, 33)):
        assert p(*dims, 0) == q(*dims, 0) and p(*dims, 1) == q(*dims, 1)
    fake = ctypes.c_void_p(0x1000)
    assert L.spin_beaver_matmul(2, 1, 4096, 4096, 4096, fake, fake, fake, fake, fake, fake, 0, fake, 16, None) == 3
