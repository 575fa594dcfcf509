// Compile-time sparsity pattern of the real tensor T[k1][k2][k3] (Sec. 3.2 eq.
// generalized_gaunt through the real basis of eq. real_swsh, App. C): the entries that the
// selection rules allow, for kernels that are unrolled over them.
//
// A real basis function (s, l, k) is a combination of complex (s, m) components: (s, |k|) and (-s, -|k|) for k != 0; one component at k = 0, both signs of s
// there in the paired basis; both blocks' components in the parity basis.  An entry needs a
// combination of components with s1 + s2 = s3, m1 + m2 = m3 whose two 3j symbols are not zero
// by symmetry (odd l1 + l2 + l3 with two equal columns or all-zero lower row), and a real
// coefficient: an even number of the functions that carry a factor i (k < 0; k = 0, s < 0 in
// the paired basis), and in the parity basis the product of the parities +1 and an even
// number of the k = 0 functions that are odd under conjugation.  For the shapes it is used
// for the rule gives exactly the nonzero entries (2,003, 2,015 and 1,535 at degree 2 with spins
// {-2..2} in the paper, paired and parity basis).
#pragma once

#include <array>
#include <cstddef>
#include <cstdint>

namespace spingtp {
namespace pattern {

enum Basis { kPaper = 0, kPaired = 1, kParity = 2 };

constexpr int abs_(int v) { return v < 0 ? -v : v; }

// One real basis function: its degree (-1: no such function, l < |s|), its components, and
// what the selection rules need of it.
struct Function {
    int l, n;          // degree, number of components
    int s[4], m[4];    // their spins and orders
    bool imag;         // carries a factor i
    bool odd_conj;     // parity basis, k = 0: odd under conjugation
    int parity;        // parity basis: +-1 (1 otherwise)
};

constexpr Function function_of(int L, int smax, int q, int basis) {
    const int block = (L + 1) * (L + 1);
    const int s = q / block - smax, r = q % block;
    int l = 0;
    while ((l + 1) * (l + 1) <= r) ++l;
    const int k = r - l * l - l, a = abs_(k);
    const int even_l = (l & 1) ? -1 : 1;
    Function f{l < abs_(s) ? -1 : l, 0, {}, {}, false, false, 1};
    const bool both_spins = basis == kParity && s != 0;
    const bool both = a != 0 || (s != 0 && basis == kPaired) || both_spins;
    for (int c = 0; c < (both_spins && a != 0 ? 4 : (both ? 2 : 1)); ++c) {
        const int e = (c & 1) ? -1 : 1;                  // (s, a) and (-s, -a)
        const int d = (c & 2) || (both_spins && a == 0 && e < 0) ? -1 : 1;  // the other block's spin
        f.s[f.n] = both_spins && a == 0 ? s * e : s * d * e;
        f.m[f.n] = a * e;
        ++f.n;
    }
    f.imag = k < 0 || (k == 0 && s < 0 && basis == kPaired);
    if (basis == kParity) {
        f.parity = s == 0 ? even_l : (s < 0 ? 1 : -1);
        f.odd_conj = k == 0 && s != 0 && (s < 0 ? 1 : -1) * even_l * ((abs_(s) & 1) ? -1 : 1) < 0;
    }
    return f;
}

// whether the entry of the functions f, g of the inputs and h of the output may be nonzero
constexpr bool allowed(const Function& f, const Function& g, const Function& h) {
    if (f.l < 0 || g.l < 0 || h.l < 0) return false;
    if (h.l < abs_(f.l - g.l) || h.l > f.l + g.l) return false;
    if ((f.imag != g.imag) != h.imag || f.parity * g.parity * h.parity < 0) return false;
    if ((f.odd_conj != g.odd_conj) != h.odd_conj) return false;
    const bool odd = ((f.l + g.l + h.l) & 1) != 0;
    for (int a = 0; a < f.n; ++a)
        for (int b = 0; b < g.n; ++b)
            for (int c = 0; c < h.n; ++c) {
                if (f.s[a] + g.s[b] != h.s[c] || f.m[a] + g.m[b] != h.m[c]) continue;
                bool zero = false;
                for (int r = 0; odd && r < 2; ++r) {  // the lower rows (m1, m2, -m3), (s1, s2, -s3)
                    const int x = r ? f.s[a] : f.m[a], y = r ? g.s[b] : g.m[b], z = -(x + y);
                    if ((x == 0 && y == 0) || (f.l == g.l && x == y) || (f.l == h.l && x == z) ||
                        (g.l == h.l && y == z))
                        zero = true;
                }
                if (!zero) return true;
            }
    return false;
}

// One term: out[o] += value A[a] B[b]; half: which of the output's two partial sums it joins
// (alternating, so that each sum is half as long).
struct Entry {
    uint8_t a, b, o, half;
};

// The entries of a square shape L1 = L2 = Lout = L.  ROLE 0 (forward): A = x1, B = x2, out;
// ROLE 1: A = grad_out, B = x2, grad_x1, and, since the product is symmetric in its inputs,
// also A = grad_out, B = x1, grad_x2.  By (a, b), then o, ascending.
template <int L, int SMAX, int BASIS, int ROLE>
struct Pattern {
    static constexpr int N = (2 * SMAX + 1) * (L + 1) * (L + 1);
    static constexpr int MAX = 2048;
    struct List {
        int n;
        Entry e[MAX];
    };
    static constexpr List make() {
        List r{};
        Function f[N] = {};
        uint8_t half[N] = {};
        for (int q = 0; q < N; ++q) f[q] = function_of(L, SMAX, q, BASIS);
        for (int a = 0; a < N; ++a)
            for (int b = 0; b < N; ++b)
                for (int o = 0; o < N; ++o) {
                    if (!(ROLE == 0 ? allowed(f[a], f[b], f[o]) : allowed(f[o], f[b], f[a]))) continue;
                    r.e[r.n] = Entry{static_cast<uint8_t>(a), static_cast<uint8_t>(b), static_cast<uint8_t>(o), half[o]};
                    half[o] ^= 1;
                    ++r.n;
                }
        return r;
    }
    static constexpr List list = make();
};

}  // namespace pattern
}  // namespace spingtp
