"""spin_completed_square_trunc against the five calls it replaces (each compared with the oracle in its own test): every
party count, odd and single-element lengths, the streaming size, the ends of the truncation range, in place on an input."""
import ctypes

import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu


def uniform(g, *shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)


@pytest.mark.parametrize("n,count,f", [(1, 1, (14, 20)), (2, 257, (1, 61)), (3, 1000, (61, 1)), (4, 4097, (16, 22)), (5, 333, (14, 20)),
                                       (6, 255, (14, 20)), (7, 256, (14, 20)), (8, 511, (14, 20)), (2, (1 << 22) + 3, (14, 20))])
def test_equals_the_separate_calls(n, count, f):
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 1000 + count)
    x = uniform(g, n, count)
    triples = [tuple(uniform(g, n, count) for _ in range(3)) for _ in range(2)]
    tuples = [tuple(uniform(g, n, count) for _ in range(3)) for _ in range(2)]
    t3, t2, lin, t0 = 2 ** 63 + 12345, 77 << 14, 2 ** 64 - 9, 5 << 28
    u = spin.lincomb_trunc([x], [1], t3)
    v = spin.lincomb_trunc([spin.beaver_mul_trunc(u, u, *triples[0], *tuples[0], f[0])], [1], t2)
    want = spin.lincomb_trunc([spin.beaver_mul(v, v, *triples[1]), x], [1, lin], t0, f[1], tuples[1])
    assert torch.equal(spin.completed_square_trunc(x, t3, t2, lin, t0, triples, tuples, f), want)
    target = tuples[1][2]
    spin.completed_square_trunc(x, t3, t2, lin, t0, triples, tuples, f, out=target)
    assert torch.equal(target, want)


def test_refusals():
    L = spin.lib()
    ok = (ctypes.c_void_p * 6)(*[0x1000] * 6)
    bad = (ctypes.c_void_p * 6)(*[0x1000] * 5 + [0x1004])
    f = lambda a, b: (ctypes.c_int * 2)(a, b)
    call = L.spin_completed_square_trunc
    assert call(2, 8, 0x1000, 0, 0, 0, 0, ok, bad, f(14, 20), 0x1000, None) == 1
    assert call(2, 8, 0x1000, 0, 0, 0, 0, None, ok, f(14, 20), 0x1000, None) == 1
    assert call(2, 8, 0x1000, 0, 0, 0, 0, ok, ok, f(0, 20), 0x1000, None) == 1
    assert call(2, 8, 0x1000, 0, 0, 0, 0, ok, ok, f(14, 62), 0x1000, None) == 1
    assert call(9, 8, 0x1000, 0, 0, 0, 0, ok, ok, f(14, 20), 0x1000, None) == 1
    assert call(2, 1 << 40, 0x1000, 0, 0, 0, 0, ok, ok, f(14, 20), 0x1000, None) == 2
