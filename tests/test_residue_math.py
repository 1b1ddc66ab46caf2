"""The arithmetic the residue GEMM relies on, replayed with Python integers from the moduli and limits written in
residue_tables.hpp: the moduli are pairwise coprime, the largest sum of one launch stays inside the range the
reconstruction tells apart, the quotient's fixed-point rounding stays inside its margin, and digits -> residues -> int32
sums -> bytes -> word gives the product mod 2^64 and 2^128, extreme operands included."""
import math
import os
import random
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_02320_amd", "csrc",
                   "residue_tables.hpp")
TEXT = open(SRC).read()
MODULI = [int(v) for v in re.search(r"kModuli\[kModuliMax\] = \{([^}]*)\}", TEXT).group(1).replace("\n", " ").split(",")]
RINGS = {bits: tuple(int(v) for v in re.search(r"ResidueRing<u%d> \{ static constexpr int L = (\d+), max_k = (\d+)" % bits,
                                               TEXT).groups()) for bits in (64, 128)}


def balanced(v, p):
    v %= p
    return v - p if 2 * v > p else v


def digits(a, bits):
    t = (a + int("80" * (bits // 8), 16)) % (1 << bits)
    return [((t >> (8 * i)) & 255) - 128 for i in range(bits // 8)]


@pytest.mark.parametrize("bits", [64, 128])
def test_moduli_and_margins(bits):
    L, max_k = RINGS[bits]
    ps = MODULI[:L]
    assert len(MODULI) == 36 and all(64 < p <= 256 for p in ps) and max_k % 64 == 0
    assert all(math.gcd(p, q) == 1 for i, p in enumerate(ps) for q in ps[:i])
    P = math.prod(ps)
    amax = 128 * (256 ** (bits // 8) - 1) // 255
    largest = 2 * max_k * amax * amax                       # 2 K products of balanced-digit integers
    frac_bits = 15 if bits == 64 else 22
    rounding = sum(255 * abs(((1 << frac_bits) + p // 2) // p - (1 << frac_bits) / p) for p in ps) / (1 << frac_bits)
    assert largest / P + rounding < 0.5
    assert 2 * max_k * 128 * 128 < 2 ** 28                   # int32 sums, with room for the reciprocal's error below
    for p in ps:
        shift = 6 if p > 128 else 5
        recip = ((1 << (32 + shift)) + p // 2) // p
        assert recip < 2 ** 31 and abs(recip * p - (1 << (32 + shift))) * 2 ** 28 / p < (1 << (32 + shift)) / p
        nd = bits // 8
        offset = 128 + p * -(-nd * 128 * 128 // p)
        r32 = -(-(1 << 32) // p)
        top = offset + nd * 128 * 128                        # the reciprocal gives the exact quotient up to here
        assert offset >= nd * 128 * 128 and all(u * r32 >> 32 == u // p for u in range(top - 2 * p, top + 1))
        assert top * (r32 * p - (1 << 32)) < 1 << 32


def word_by_residues(terms, bits):
    L, _ = RINGS[bits]
    ps, nd = MODULI[:L], bits // 8
    P = math.prod(ps)
    ys = []
    for p in ps:
        inv = pow(P // p, -1, p)
        left = [balanced(256 ** i, p) for i in range(nd)]
        right = [balanced(256 ** i * inv, p) for i in range(nd)]
        offset = 128 + p * -(-nd * 128 * 128 // p)
        acc = 0
        for a, b in terms:
            x = (sum(s * w for s, w in zip(digits(a, bits), left)) + offset) % p - 128
            y = (sum(s * w for s, w in zip(digits(b, bits), right)) + offset) % p - 128
            assert -128 <= x < 128 and -128 <= y < 128
            acc += x * y
        shift = 6 if p > 128 else 5
        q = (acc * (((1 << (32 + shift)) + p // 2) // p)) >> (32 + shift)
        assert 0 <= acc - q * p <= p
        ys.append((acc - q * p) & 255)
    frac_bits = 15 if bits == 64 else 22
    Q = (sum(y * (((1 << frac_bits) + p // 2) // p) for y, p in zip(ys, ps)) + (1 << (frac_bits - 1))) >> frac_bits
    assert Q < 256
    return (sum(y * (P // p) for y, p in zip(ys, ps)) - Q * P) % (1 << bits)


@pytest.mark.parametrize("bits", [64, 128])
def test_word_from_residues(bits):
    rng = random.Random(bits)
    M = 1 << bits
    low = int("80" * (bits // 8), 16)                        # every digit -128
    high = int("7f" * (bits // 8), 16)
    cases = [[(low, low)] * 40, [(high, high)] * 40, [(low, high)] * 40, [(0, 0)], [(M - 1, 1)], [(M // 2, M // 2)] * 9]
    cases += [[(rng.randrange(M), rng.randrange(M)) for _ in range(rng.randint(1, 40))] for _ in range(40)]
    for terms in cases:
        assert word_by_residues(terms, bits) == sum(a * b for a, b in terms) % M


# The choice by estimate shows in the preferred workspace: above the required one only where the residue GEMM is taken.
# Batched, long and narrow-tiled products near the line, whose estimates once fell on the wrong side, and clear ones.
@pytest.mark.parametrize("dims,residue", [((3, 2, 700, 700, 700), False), ((4, 1, 4096, 200, 2048), False),
                                          ((5, 1, 512, 512, 512), False), ((2, 1, 64, 64, 64), False),
                                          ((2, 1, 2048, 2048, 2048), True), ((5, 1, 4096, 4096, 4096), True)])
def test_choice_near_the_line(dims, residue):
    from paper_2402_02320_amd import spin
    L = spin.lib()
    need = L.spin_beaver_matmul_workspace_bytes(*dims, spin.LIMB_MFMA)
    assert (L.spin_beaver_matmul_preferred_workspace_bytes(*dims, spin.LIMB_MFMA) > need) is residue
