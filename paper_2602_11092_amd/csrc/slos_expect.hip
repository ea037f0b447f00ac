// Per-mode photon-number expectations over the full Fock space, without the
// Fock space (arXiv 2602.11092, Sec. II-B measurement strategies).
//
// With V the n columns of U that carry the photons and phi_i the state without
// photon i, removing a photon from mode j gives a_j |psi> = sum_i V[j][i] |phi_i>, so
//
//     <n_j> = ||a_j psi||^2 = (1 / prod s!) sum_{a,b} conj(V[j][a]) V[j][b] P_ab,
//
// P_ab = <phi_a|phi_b> = Perm of G = V^H V without row a and column b
// (Cauchy-Binet over all outputs, for any V, unitary or not).  For the
// gradient, L = sum_j w_j <n_j> = (1 / prod s!) d/de Perm(G + e E) at e = 0 with
// E_ab = sum_j w_j conj(V[j][a]) V[j][b], so with D_ab = d/de P_ab(G + e E)
//
//     dL/dV[j][a] = (2 / prod s!) sum_b (w_j P_ab + D_ab) V[j][b].
//
// All P_ab come from permanents of the first rows over every subset of
// columns and of the last rows over every subset (n 2^(n-1) products each); the
// adjoint carries (value, e-derivative) pairs through the same sums.  n = 5
// takes 240 products where the photon recursion takes 252000 at m = 20.
// FP64 (the sums are tiny), one wave per sample: bound by the latency of its
// 2 n short steps.  m = 20, n = 5, B = 512: forward 11 us, adjoint 26 us; the
// recursion with the expectation epilogue took 103 us, and the expanded weights
// and the probability adjoint 229 us.
#include "slos_internal.h"

namespace slos {
namespace {

constexpr int kExpMaxN = 8;  // 2^8 subsets of pairs of complex FP64 values, 16 KB of LDS

__device__ __forceinline__ void z_fma(double2& acc, double2 a, double2 b) {
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(-a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(a.y, b.x, acc.y);
}
__device__ __forceinline__ void z_fma_conj(double2& acc, double2 a, double2 b) {  // acc += conj(a) b
    z_fma(acc, make_double2(a.x, -a.y), b);
}

template <bool BWD>
__global__ __launch_bounds__(64) void expect_closed_kernel(int m, BatchDev Bt, const float2* __restrict__ U,
                                                           const float* __restrict__ w, float* __restrict__ out,
                                                           float2* __restrict__ gU) {
    constexpr int H = BWD ? 2 : 1;  // values, and their e-derivatives
    __shared__ double2 V[kMaxModes * kExpMaxN];
    __shared__ double2 M[H][kExpMaxN * kExpMaxN];           // G and E, row a, column b
    __shared__ double2 F[H][1 << kExpMaxN], L[H][1 << kExpMaxN];  // first rows, last rows, by column subset
    __shared__ double2 P[H][kExpMaxN * kExpMaxN];
    const int lane = threadIdx.x, b = blockIdx.x;
    const int n = ldc(Bt.n + b);
    const float2* Ub = U + (size_t)b * m * m;
    if (n == 0) {  // the vacuum: <n_j> = 0 for every U
        if (!BWD) {
            if (lane < m) out[(size_t)b * m + lane] = 0.f;
        } else {
            for (int e = lane; e < m * m; e += 64) gU[(size_t)b * m * m + e] = c_zero();
        }
        return;
    }
    int mode[kExpMaxN];
    double scale = 1.0;
    int run = 1;
#pragma unroll
    for (int i = 0; i < kExpMaxN; ++i) {
        mode[i] = i < n ? ldc(Bt.modes + (size_t)b * kMaxPhotons + i) : -1;
        run = i > 0 && mode[i] == mode[i > 0 ? i - 1 : 0] ? run + 1 : 1;
        if (i < n) scale /= run;
    }
    for (int e = lane; e < m * n; e += 64) {
        const int j = e / n, i = e % n;
        const float2 v = Ub[j * m + ldg(Bt.modes + (size_t)b * kMaxPhotons + i)];
        V[e] = make_double2(v.x, v.y);
    }
    __syncthreads();
    if (lane < n * n) {
        const int a = lane / n, c = lane % n;
        double2 g = make_double2(0.0, 0.0), e = g;
        for (int j = 0; j < m; ++j) {
            double2 t = make_double2(0.0, 0.0);
            z_fma_conj(t, V[j * n + a], V[j * n + c]);
            g.x += t.x;
            g.y += t.y;
            if (BWD) {
                const double wj = w[(size_t)b * m + j];
                e.x = fma(wj, t.x, e.x);
                e.y = fma(wj, t.y, e.y);
            }
        }
        M[0][lane] = g;
        if (BWD) M[H - 1][lane] = e;
    }
    if (lane == 0) {
        F[0][0] = L[0][0] = make_double2(1.0, 0.0);
        if (BWD) F[H - 1][0] = L[H - 1][0] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    const int full = (1 << n) - 1;
    for (int l = 1; l < n; ++l) {  // minors leave one row out: subsets of up to n-1 columns
        const int rf = (l - 1) * n, rl = (n - l) * n;
        for (int s = lane; s <= full; s += 64) {
            if (__builtin_popcount(s) != l) continue;
            double2 f = make_double2(0.0, 0.0), fe = f, q = f, qe = f;
            for (int i = 0; i < n; ++i) {
                if (!((s >> i) & 1)) continue;
                const int r = s & ~(1 << i);
                z_fma(f, M[0][rf + i], F[0][r]);
                z_fma(q, M[0][rl + i], L[0][r]);
                if (BWD) {
                    z_fma(fe, M[0][rf + i], F[H - 1][r]);
                    z_fma(fe, M[H - 1][rf + i], F[0][r]);
                    z_fma(qe, M[0][rl + i], L[H - 1][r]);
                    z_fma(qe, M[H - 1][rl + i], L[0][r]);
                }
            }
            F[0][s] = f;
            L[0][s] = q;
            if (BWD) {
                F[H - 1][s] = fe;
                L[H - 1][s] = qe;
            }
        }
        __syncthreads();
    }
    if (lane < n * n) {  // rows before a take the columns s, rows after it the rest but column c
        const int a = lane / n, c = lane % n;
        double2 p = make_double2(0.0, 0.0), d = p;
        for (int s = 0; s <= full; ++s) {
            if (__builtin_popcount(s) != a || ((s >> c) & 1)) continue;
            const int r = full & ~s & ~(1 << c);
            z_fma(p, F[0][s], L[0][r]);
            if (BWD) {
                z_fma(d, F[0][s], L[H - 1][r]);
                z_fma(d, F[H - 1][s], L[0][r]);
            }
        }
        P[0][lane] = p;
        if (BWD) P[H - 1][lane] = d;
    }
    __syncthreads();
    if constexpr (!BWD) {
        if (lane < m) {
            double v = 0.0;
            for (int a = 0; a < n; ++a) {
                double2 t = make_double2(0.0, 0.0);
                for (int c = 0; c < n; ++c) z_fma(t, P[0][a * n + c], V[lane * n + c]);
                v += V[lane * n + a].x * t.x + V[lane * n + a].y * t.y;
            }
            out[(size_t)b * m + lane] = (float)(scale * v);
        }
    } else {
        for (int e = lane; e < m * m; e += 64) {
            const int j = e / m, col = e % m;
            const double wj = w[(size_t)b * m + j];
            double2 g = make_double2(0.0, 0.0);
            for (int a = 0; a < n; ++a) {
                if (ldg(Bt.modes + (size_t)b * kMaxPhotons + a) != col) continue;
                for (int c = 0; c < n; ++c) {
                    const double2 p = P[0][a * n + c], d = P[H - 1][a * n + c];
                    z_fma(g, make_double2(fma(wj, p.x, d.x), fma(wj, p.y, d.y)), V[j * n + c]);
                }
            }
            gU[(size_t)b * m * m + e] = make_float2((float)(2.0 * scale * g.x), (float)(2.0 * scale * g.y));
        }
    }
}

}  // namespace

// The full Fock space only (a restricted one is not all of Cauchy-Binet's
// outputs), and photon numbers whose subset tables fit LDS.
bool expect_closed_ok(const slos_batch_s& Bt) { return !restricted_plan(*Bt.plan) && Bt.n_max <= kExpMaxN; }

int launch_expect_closed(const slos_batch_s& Bt, bool bwd, const float2* U, const float* w, float* out, float2* gU,
                         hipStream_t stream) {
    void* fn = bwd ? (void*)&expect_closed_kernel<true> : (void*)&expect_closed_kernel<false>;
    void* args[] = {(void*)&Bt.plan->m, (void*)&Bt.dev, (void*)&U, (void*)&w, (void*)&out, (void*)&gU};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)Bt.B), dim3(64), args, 0, stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("expectation launch: ") + hipGetErrorString(e));
    return SLOS_OK;
}

}  // namespace slos
