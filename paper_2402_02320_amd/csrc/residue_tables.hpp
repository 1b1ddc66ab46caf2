// Constants of the residue-number GEMM (gemm_residue.hip): pairwise coprime moduli of at most eight bits and what
// follows from them by modular arithmetic, all computed at compile time.
//
// A ring element a of ND bytes is the integer a' = sum_i s_i 256^i of its balanced digits s_i in [-128,127]
// (a' == a mod 2^(8 ND), |a'| <= 128 (256^ND - 1) / 255).  The integer S = sum of the products of an output element
// is determined by its residues modulo L pairwise coprime p_l as long as |S| < P / 2, P = prod p_l:
//     y_l = S (P/p_l)^-1 mod p_l,     S = sum_l y_l (P/p_l) - Q P,     Q = round(sum_l y_l / p_l).
// The moduli are the set of at most eight bits each with the largest product found for 36 members; its first 18
// members are the best set of 18.
#pragma once
#include "common.hpp"

namespace spin {
namespace {

constexpr int kModuliMax = 36;
constexpr int kModuli[kModuliMax] = {256, 253, 251, 249, 247, 241, 239, 235, 233, 229, 227, 223,
                                     217, 211, 199, 197, 193, 191, 181, 179, 173, 167, 163, 157,
                                     151, 149, 139, 137, 131, 127, 113, 109, 107, 103, 101, 97};

template <class T> struct ResidueRing;
// max_k: the longest inner dimension K of one launch (two products per output element, 2 K terms): with
// |S| <= 2 K amax^2 <= 0.40 P the fraction of S/P stays 0.10 away from the rounding boundary of Q.  A multiple of 64.
template <> struct ResidueRing<u64> { static constexpr int L = 18, max_k = 5632; };
template <> struct ResidueRing<u128> { static constexpr int L = 36, max_k = 3712; };

constexpr int mod_pow256(int e, int p)
{
    int r = 1 % p;
    for (int i = 0; i < e; ++i) r = (int)((long)r * 256 % p);
    return r;
}
constexpr int balanced(int v, int p) { return 2 * v > p ? v - p : v; }
constexpr u32 byte_at(int v, int pos) { return (u32)(v & 255) << (8 * pos); }

template <class T> struct ResidueTables {
    static constexpr int L = ResidueRing<T>::L, ND = sizeof(T), NW = ND / 4;
    static constexpr int groups = (L + 1 + 3) / 4;       // of four bytes: L residues and Q
    // conversion: weights of the digits (four to a word); right operands carry the factor (P/p_l)^-1
    u32 left[L][NW], right[L][NW];
    u32 offset[L];                                       // == 128 (mod p), makes every weighted digit sum non-negative
    u32 recip[L];                                        // ceil(2^32 / p)
    // reduction of an int32 accumulator: q = floor(acc * acc_recip / 2^(32 + acc_shift)) = floor(acc / p)
    int acc_recip[L], acc_shift[L];
    // reconstruction: byte j of P/p_l (and of -P in the slot of Q), four moduli to a word; 1/p_l in fixed point
    u32 weight[ND][groups];
    // With one byte per modulus (every p_l > 128) the 18 roundings of 2^15 / p_l move sum_l y_l / p_l by at most 0.037,
    // inside the 0.10 that max_k leaves; with smaller moduli a second byte is needed.
    static constexpr bool two_level = ND == 16;
    static constexpr int frac_bits = two_level ? 22 : 15;
    u32 frac_hi[groups], frac_lo[groups];                // two_level: 2^22 / p_l = 256 frac_hi + frac_lo; else 2^15 / p_l

    constexpr ResidueTables()
        : left{}, right{}, offset{}, recip{}, acc_recip{}, acc_shift{}, weight{}, frac_hi{}, frac_lo{}
    {
        T all = 1;
        for (int l = 0; l < L; ++l) all = all * (T)kModuli[l];
        for (int l = 0; l < L; ++l) {
            const int p = kModuli[l];
            int others_p = 1;                            // P / p_l mod p_l
            T others = 1;                                // P / p_l mod 2^(8 ND)
            for (int m = 0; m < L; ++m)
                if (m != l) {
                    others_p = (int)((long)others_p * kModuli[m] % p);
                    others = others * (T)kModuli[m];
                }
            int inv = 1;
            while ((long)inv * others_p % p != 1) ++inv;
            for (int i = 0; i < ND; ++i) {
                const int w = mod_pow256(i, p);
                left[l][i / 4] |= byte_at(balanced(w, p), i % 4);
                right[l][i / 4] |= byte_at(balanced((int)((long)w * inv % p), p), i % 4);
            }
            offset[l] = 128 + (u32)p * ((ND * 128 * 128 + (u32)p - 1) / (u32)p);
            recip[l] = (u32)((0x100000000ull + (u64)p - 1) / (u64)p);
            acc_shift[l] = p > 128 ? 6 : 5;
            acc_recip[l] = (int)(((1ull << (32 + acc_shift[l])) + (u64)p / 2) / (u64)p);
            for (int j = 0; j < ND; ++j) weight[j][l / 4] |= byte_at((int)((others >> (8 * j)) & 255), l % 4);
            const u32 f = ((1u << frac_bits) + (u32)p / 2) / (u32)p;
            frac_hi[l / 4] |= (two_level ? f >> 8 : f) << (8 * (l % 4));
            frac_lo[l / 4] |= (f & 255) << (8 * (l % 4));
        }
        const T minus = (T)0 - all;
        for (int j = 0; j < ND; ++j) weight[j][L / 4] |= byte_at((int)((minus >> (8 * j)) & 255), L % 4);
    }
};
template <class T> inline constexpr ResidueTables<T> kResidue{};

}  // namespace
}  // namespace spin
