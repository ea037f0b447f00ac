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
// FP64 (the sums are tiny).  Bound by the latency of its n dependent levels, hence
// a thread per column subset (a workgroup of 64 up to 6 photons, 256 for 7 and 8), and
// four threads per matrix entry in the wide one.  One wave with loops over all
// subsets took 44 us for a sample of 8 photons, which lost to the photon recursion
// wherever the Fock space is small.  us, forward / adjoint, the recursion (the
// adjoint from expanded weights) and here: m = 20, n = 5, B = 512 94 / 214 and 7.5 /
// 13.6; m = 6, n = 8 (1287 states) B = 1 15 / 32 and 9.9 / 13.9, B = 8192 123 / 329 and
// 70 / 121; m = 3, n = 8 (45 states) B = 1 12 / 22 and 9.7 / 14, B = 1024 13.3 / 42 and
// 14.8 / 23; m = 2, n = 3 (4 states) B = 1 8.2 / 10.9 and 5.6 / 5.8.
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

// Sum over the S adjacent lanes that share an entry.
template <int S>
__device__ __forceinline__ double2 share_sum(double2 v) {
    for (int s = 1; s < S; s <<= 1) {
        v.x += __shfl_xor(v.x, s, 64);
        v.y += __shfl_xor(v.y, s, 64);
    }
    return v;
}

// NT threads, one per subset of the columns: 64 up to 6 photons, 256 for 7 and 8.
template <bool BWD, int NT>
__global__ __launch_bounds__(NT) void expect_closed_kernel(int m, BatchDev Bt, const float2* __restrict__ U,
                                                           const float* __restrict__ w, float* __restrict__ out,
                                                           float2* __restrict__ gU) {
    constexpr int H = BWD ? 2 : 1;  // values, and their e-derivatives
    constexpr int S = NT / 64;      // threads that share an entry of an 8 x 8 matrix
    // matrices and V in rows of eight: indexes by shifts
    __shared__ double2 V[kMaxModes * 8];
    __shared__ double2 M[H][64];          // G and E, row a, column b
    __shared__ double2 F[H][NT], L[H][NT];  // first rows, last rows, by column subset
    __shared__ double2 P[H][64];
    __shared__ int mode[8];
    const int tid = threadIdx.x;
    const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (b >= Bt.B) return;
    const int n = ldc(Bt.n + b);
    const float2* Ub = U + b * m * m;
    if (n == 0) {  // the vacuum: <n_j> = 0 for every U
        if (!BWD) {
            if (tid < m) out[b * m + tid] = 0.f;
        } else {
            for (int e = tid; e < m * m; e += NT) gU[b * m * m + e] = c_zero();
        }
        return;
    }
    {
        const int i = tid & 7;
        const int mi = ldg(Bt.modes + b * kMaxPhotons + i);
        if (tid < 8) mode[i] = i < n ? mi : -1;
        for (int j = tid >> 3; j < m; j += NT / 8) {
            const float2 v = i < n ? Ub[j * m + mi] : c_zero();
            V[8 * j + i] = make_double2(v.x, v.y);
        }
    }
    if (tid == 0) {
        F[0][0] = L[0][0] = make_double2(1.0, 0.0);
        if (BWD) F[H - 1][0] = L[H - 1][0] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    double scale = 1.0;
    for (int i = 1, run = 1; i < n; ++i) {
        run = mode[i] == mode[i - 1] ? run + 1 : 1;
        scale /= run;
    }
    // entry (a, c) of the matrices, share q of its sums
    const int a = tid / (8 * S), c = tid / S & 7, q = tid % S;
    {
        double2 g = make_double2(0.0, 0.0), e = g;
#pragma unroll 4
        for (int j = q; j < m; j += S) {
            double2 t = make_double2(0.0, 0.0);
            z_fma_conj(t, V[8 * j + a], V[8 * j + c]);
            g.x += t.x;
            g.y += t.y;
            if (BWD) {
                const double wj = w[b * m + j];
                e.x = fma(wj, t.x, e.x);
                e.y = fma(wj, t.y, e.y);
            }
        }
        g = share_sum<S>(g);
        if (BWD) e = share_sum<S>(e);
        if (q == 0) {
            M[0][8 * a + c] = g;
            if (BWD) M[H - 1][8 * a + c] = e;
        }
    }
    __syncthreads();
    const int full = (1 << n) - 1, size = tid <= full ? __builtin_popcount(tid) : 0;
    for (int l = 1; l < n; ++l) {  // minors leave one row out: subsets of up to n-1 columns
        if (size == l) {
            const int rf = 8 * (l - 1), rl = 8 * (n - l);
            double2 f = make_double2(0.0, 0.0), fe = f, p = f, pe = f;
            for (int left = tid; left != 0; left &= left - 1) {
                const int i = __builtin_ctz(left), r = tid & ~(1 << i);
                z_fma(f, M[0][rf + i], F[0][r]);
                z_fma(p, M[0][rl + i], L[0][r]);
                if (BWD) {
                    z_fma(fe, M[0][rf + i], F[H - 1][r]);
                    z_fma(fe, M[H - 1][rf + i], F[0][r]);
                    z_fma(pe, M[0][rl + i], L[H - 1][r]);
                    z_fma(pe, M[H - 1][rl + i], L[0][r]);
                }
            }
            F[0][tid] = f;
            L[0][tid] = p;
            if (BWD) {
                F[H - 1][tid] = fe;
                L[H - 1][tid] = pe;
            }
        }
        __syncthreads();
    }
    {  // rows before a take the columns s, rows after it the rest but column c: the
       // n-1 other columns' subsets r of size a
        double2 p = make_double2(0.0, 0.0), d = p;
        if (a < n && c < n) {
#pragma unroll 4
            for (int r = q; r < 1 << (n - 1); r += S) {
                if (__builtin_popcount(r) != a) continue;
                const int s = (r & ((1 << c) - 1)) | (r >> c) << (c + 1), rest = full & ~s & ~(1 << c);
                z_fma(p, F[0][s], L[0][rest]);
                if (BWD) {
                    z_fma(d, F[0][s], L[H - 1][rest]);
                    z_fma(d, F[H - 1][s], L[0][rest]);
                }
            }
        }
        p = share_sum<S>(p);
        if (BWD) d = share_sum<S>(d);
        if (q == 0) {
            P[0][8 * a + c] = p;
            if (BWD) P[H - 1][8 * a + c] = d;
        }
    }
    __syncthreads();
    // thread (j, row): row of P V for mode j
    const int row = tid & 7;
    for (int j0 = 0; j0 < m; j0 += NT / 8) {
        const int j = j0 + (tid >> 3);
        double2 t = make_double2(0.0, 0.0);
        if (j < m && row < n) {
            const double wj = BWD ? w[b * m + j] : 0.0;
            for (int i = 0; i < n; ++i) {
                const double2 p = P[0][8 * row + i];
                if (BWD) {
                    const double2 d = P[H - 1][8 * row + i];
                    z_fma(t, make_double2(fma(wj, p.x, d.x), fma(wj, p.y, d.y)), V[8 * j + i]);
                } else {
                    z_fma(t, p, V[8 * j + i]);
                }
            }
        }
        if constexpr (!BWD) {
            double v = j < m && row < n ? V[8 * j + row].x * t.x + V[8 * j + row].y * t.y : 0.0;
            for (int s = 1; s < 8; s <<= 1) v += __shfl_xor(v, s, 64);
            if (j < m && row == 0) out[b * m + j] = (float)(scale * v);
        } else {
            __syncthreads();  // gradients of NT / 8 modes at a time through F
            F[0][tid] = t;
            __syncthreads();
            const int rows = min(m - j0, NT / 8);
            for (int e = tid; e < rows * m; e += NT) {
                const int jj = e / m, col = e % m;
                double2 g = make_double2(0.0, 0.0);
                for (int i = 0; i < n; ++i)
                    if (mode[i] == col) {
                        g.x += F[0][8 * jj + i].x;
                        g.y += F[0][8 * jj + i].y;
                    }
                gU[b * m * m + (int64_t)j0 * m + e] = make_float2((float)(2.0 * scale * g.x), (float)(2.0 * scale * g.y));
            }
        }
    }
}

}  // namespace

// The full Fock space only (a restricted one is not all of Cauchy-Binet's
// outputs), and photon numbers whose subset tables fit LDS.
bool expect_closed_ok(const slos_batch_s& Bt) { return !restricted_plan(*Bt.plan) && Bt.n_max <= kExpMaxN; }

int launch_expect_closed(const slos_batch_s& Bt, bool bwd, const float2* U, const float* w, float* out, float2* gU,
                         hipStream_t stream) {
    const bool wide = Bt.n_max > 6;
    void* fn = bwd ? (wide ? (void*)&expect_closed_kernel<true, 256> : (void*)&expect_closed_kernel<true, 64>)
                   : (wide ? (void*)&expect_closed_kernel<false, 256> : (void*)&expect_closed_kernel<false, 64>);
    void* args[] = {(void*)&Bt.plan->m, (void*)&Bt.dev, (void*)&U, (void*)&w, (void*)&out, (void*)&gU};
    // (a dimension of a launch holds less than 2^32 threads)
    const unsigned gx = std::min((unsigned)Bt.B, 1u << 22), gy = ((unsigned)Bt.B + gx - 1) / gx;
    hipError_t e = hipLaunchKernel(fn, dim3(gx, gy), dim3(wide ? 256 : 64), args, 0, stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("expectation launch: ") + hipGetErrorString(e));
    return SLOS_OK;
}

}  // namespace slos
