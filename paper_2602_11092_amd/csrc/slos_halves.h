// Two-halves evaluation of Fock spaces beyond on-chip memory: tables and
// compile-time subset algebra shared by the kernels of slos_halves.hip.
//
// Cut the modes into a low half [0, c) and a high half [c, m).  An output
// state is a pair (alpha, beta) of a k-photon state of the low half and an
// (n-k)-photon state of the high half, and its permanent splits by which k of
// the n input photons went low (Laplace expansion along those rows):
//
//     a(alpha, beta) = sum_{S subset of [n], |S| = k} A_k[S][alpha] B_{n-k}[S^c][beta],
//
//     A_k[S][alpha] = Perm(U[alpha, S]) / sqrt(prod alpha!),  B likewise.
//
// For each k that is a dense complex product with an inner length of C(n, k):
// no transition tables and no gathers, and matrix instructions apply.  In the
// basis order (lexicographic in the sorted mode list) the outputs of one alpha
// are contiguous in beta.  A half's factors come from its own short recursion
// over its first mode: with alpha = (j, alpha'), j <= first(alpha'),
//
//     A_k[S][alpha] = mu^(-1/2) sum_{i in S} U[j][i] A_{k-1}[S \ i][alpha'],
//
// mu = copies of j at the front of alpha.  The states with first mode j are
// contiguous, and so are the alpha' they extend (those whose first mode is
// not below j), so row -> parent row is a shift within each j.
#pragma once

#include "slos_internal.h"

namespace slos {

__host__ __device__ constexpr int sub_binom(int n, int k) {
    int r = 1;
    for (int i = 1; i <= k; ++i) r = r * (n - i + 1) / i;
    return r;
}

// Subsets of [N] by size in ascending numeric order of their masks (the
// complement of subset q of size l is subset C-1-q of size N-l), and for each
// subset S of size L its terms (i, rank of S \ i).
template <int N, int L>
struct SubsetTerms {
    static constexpr int K = sub_binom(N, L);
    int i[K][L > 0 ? L : 1] = {};
    int src[K][L > 0 ? L : 1] = {};
    constexpr SubsetTerms() {
        int q = 0;
        for (int s = 0; s < (1 << N); ++s) {
            int pc = 0;
            for (int b = 0; b < N; ++b) pc += (s >> b) & 1;
            if (pc != L) continue;
            int t = 0;
            for (int b = 0; b < N; ++b) {
                if (!((s >> b) & 1)) continue;
                const int r = s & ~(1 << b);
                int rank = 0;
                for (int x = 0; x < r; ++x) {
                    int px = 0;
                    for (int y = 0; y < N; ++y) px += (x >> y) & 1;
                    rank += px == L - 1;
                }
                i[q][t] = b;
                src[q][t] = rank;
                ++t;
            }
            ++q;
        }
    }
};

}  // namespace slos
