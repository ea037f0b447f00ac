// Dense amplitude-encoded inputs, one interferometer per input (arXiv
// 2602.11092, Sec. II-C-2): the whole superposition goes through U photon by
// photon instead of one simulation per component.
//
// With sum_s x_s |s> written as a symmetric polynomial in the input modes,
// one photon at a time is replaced by its image under U.  After k photons the
// state is T_k[J][I], J a k-photon output state and I the (n-k)-photon input
// state still to go:
//
//   T_0[s] = x_s sqrt(prod s!),
//   T_{k+1}[J + e_j][I'] = sum_i U[j][i] T_k[J][I' + e_i]   (j the first mode of J + e_j),
//   y_t = T_n[t] / sqrt(prod t!).
//
// T_k is symmetric in its output photons, so any photon of J + e_j may be the
// new one; the first is taken.  The cost is sum_k N_k N_{n-k} m products
// against N_n sum_k k N_k for one simulation per basis state (m = 6, n = 3:
// 1848 against 12432), and nothing but x, U and the result leaves the chip.
// The adjoint walks the same steps back:
//
//   gT_k[J][I] = sum_{j <= first(J)} sum_{i in I} conj(U[j][i]) gT_{k+1}[J + e_j][I - e_i],
//   gU[j][i]  += sum conj(T_k[J][I' + e_i]) gT_{k+1}[J + e_j][I']  over J with first(J) >= j and I'.
//
// The sums are FP64 and T is kept in FP32, one rounding a step; gT is carried in
// FP64, so that dL/dx (gT_0, scaled) is rounded once.  Relative error against 64 bits,
// m = 8, n = 3, 64 inputs, one simulation per component and here: y 2.2e-7 / 5.3e-8,
// dL/dU 1.5e-7 / 4.1e-8, dL/dx 8.2e-8 / 2.6e-8.  (With FP32 sums dL/dU was off by 1.8e-7.)
//
// One workgroup per input; T, gT, U and 16-bit copies of the transition
// tables sit in LDS (m = 6, n = 3: 9 KB).  The kernels are bound by the
// latency of their 2 n short steps, and overlap over the inputs of a CU.
// Fixed summation orders throughout: results are bitwise reproducible.
// Measured at m = 6, n = 3, 1024 inputs of 56 components, against one
// simulation per component: forward 10 us (195), adjoint 23 us (1092).
#include "slos_internal.h"

namespace slos {
namespace {

constexpr int kDenseBlock = 128;

// LDS plan of an n-photon input (bytes).
struct DenseLayout {
    uint32_t T[kMaxPhotons + 1];     // T_k, float2 [N_k][N_{n-k}]
    uint32_t g[2], gn;               // gT_k at g[k & 1] for k < n, and gT_n, double2 (backward)
    uint32_t U;                      // double2 [m][m], widened once
    uint32_t part;                   // double2 [kDenseBlock]: partial sums of gU (backward)
    uint32_t succ[kMaxPhotons + 1];  // uint16 [N_{l-1}][m], l = 1..n: rank of I' + e_i
    uint32_t pred[kMaxPhotons + 1];  // uint16 [N_l][l][2], l = 1..n: mode and rank of the removals, mode 0xFFFF: none
    uint32_t bytes;
};
__host__ __device__ inline void dense_layout(const int* N, int m, int n, bool bwd, DenseLayout& L) {
    uint32_t at = 0, most[2] = {0, 0};  // largest T_k, k < n, of each parity
    for (int k = 0; k <= n; ++k) {
        L.T[k] = at;
        const uint32_t b = 8u * (uint32_t)N[k] * (uint32_t)N[n - k];
        if (k < n) most[k & 1] = b > most[k & 1] ? b : most[k & 1];
        if (k < n || !bwd) at += b;  // the adjoint starts from the given gradient, not from T_n
    }
    if (bwd) {
        // gT_{n-2}, gT_{n-4}, .. are formed when T_{n-1} and gT_n have been read: over both
        L.T[n - 1] = (L.T[n - 1] + 15u) & ~15u;
        L.g[n & 1] = L.T[n - 1];
        L.gn = (L.T[n - 1] + 8u * (uint32_t)N[n - 1] * (uint32_t)N[1] + 15u) & ~15u;
        const uint32_t over = L.g[n & 1] + 2 * most[n & 1], end = L.gn + 16u * (uint32_t)N[n];
        at = ((over > end ? over : end) + 15u) & ~15u;
        L.g[(n - 1) & 1] = at;
        at += 2 * most[(n - 1) & 1];
    }
    L.part = at;
    at += bwd ? 16u * kDenseBlock : 0;
    at = (at + 15u) & ~15u;
    L.U = at;
    at += 16u * (uint32_t)(m * m);
    for (int l = 1; l <= n; ++l) {
        L.succ[l] = at;
        at += (2u * (uint32_t)(N[l - 1] * m) + 3u) & ~3u;
    }
    for (int l = 1; l <= n; ++l) {
        L.pred[l] = at;
        at += 4u * (uint32_t)(N[l] * l);
    }
    L.bytes = at;
}

struct DenseArgs {
    int m;
    const LayerDev* Ls;
    BatchDev Bt;
    const int64_t* goff;
    const int64_t* ooff;
    const int32_t* crank;    // [C] rank of the component's state
    const float* cnorm;      // [C] sqrt(prod s!)
    const uint32_t* gcols;   // [G] input modes its components use
    const float2* U;         // [G][m][m]
    const float2* x;         // [C]
    const float2* gy;        // gradient of the outputs (backward)
    float2* y;               // outputs (forward)
    float2* gU;              // [G][m][m] (backward)
    float2* gx;              // [C] or nullptr (backward)
};

__device__ __forceinline__ void z_fma_conj(double2& acc, double2 a, double2 b) {  // acc += conj(a) b
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(-a.y, b.x, acc.y);
}

// prod t! of the state whose n removals are pred (a mode's further photons are
// marked 0xFFFF).
__device__ __forceinline__ double fact_of(const uint16_t* pred, int n) {
    double f = 1.0;
    int run = 1;
    for (int q = 0; q < n; ++q) {
        run = pred[2 * q] == 0xFFFF ? run + 1 : 1;
        f *= run;
    }
    return f;
}

// T_0 .. T_{n-1} (backward) or T_n (forward) of input g in LDS, with its tables.
template <bool BWD>
__global__ __launch_bounds__(kDenseBlock) void dense_kernel(DenseArgs A) {
    extern __shared__ char dlds[];
    const int tid = threadIdx.x, g = blockIdx.x, m = A.m;
    const int64_t c0 = ldc(A.goff + g), c1 = ldc(A.goff + g + 1), o0 = ldc(A.ooff + g);
    const int n = ldc(A.Bt.n + c0);
    const uint32_t cols = ldc(A.gcols + g);
    int N[kMaxPhotons + 1];
#pragma unroll
    for (int k = 0; k <= kMaxPhotons; ++k) N[k] = k <= n ? (int)ldc(&A.Ls[k].N) : 0;
    DenseLayout L;
    dense_layout(N, m, n, BWD, L);
    double2* U = (double2*)(dlds + L.U);
    // U with the columns no component uses left out (they may hold anything)
    for (int e = tid; e < m * m; e += kDenseBlock) {
        const float2 v = (cols >> (e % m)) & 1 ? A.U[(size_t)g * m * m + e] : c_zero();
        U[e] = make_double2(v.x, v.y);
    }
    float2* T0 = (float2*)(dlds + L.T[0]);
    for (int e = tid; e < N[n]; e += kDenseBlock) T0[e] = c_zero();
    for (int l = 1; l <= n; ++l) {
        const LayerDev* P = A.Ls + l;
        const uint32_t* succ = ldc(&P->succ);
        const uint32_t* pv = (const uint32_t*)ldc(&P->predv);
        const int shift = ldc(&P->pred_shift);
        uint16_t* s = (uint16_t*)(dlds + L.succ[l]);
        for (int e = tid; e < N[l - 1] * m; e += kDenseBlock) {
            const int t = e / m, j = e % m;
            s[e] = (uint16_t)(ldg(succ + ((size_t)(j / 4) * N[l - 1] + t) * 4 + (j & 3)) >> 3);
        }
        uint16_t* p = (uint16_t*)(dlds + L.pred[l]);
        for (int e = tid; e < N[l] * l; e += kDenseBlock) {
            const int t = e / l, q = e % l;
            const uint32_t w = ldg(pv + ((size_t)(q / 4) * N[l] + t) * 4 + (q & 3));
            const uint32_t mode = w >> shift;
            p[2 * e] = (uint16_t)(mode == 32 ? 0xFFFF : mode);
            p[2 * e + 1] = (uint16_t)((w & pred_rank_mask(shift)) >> 3);
        }
    }
    __syncthreads();
    for (int64_t c = c0 + tid; c < c1; c += kDenseBlock) T0[ldg(A.crank + c)] = c_scale(A.x[c], ldg(A.cnorm + c));
    __syncthreads();
    for (int k = 0; k < (BWD ? n - 1 : n); ++k) {
        const float2* Tk = (const float2*)(dlds + L.T[k]);
        float2* Tn = (float2*)(dlds + L.T[k + 1]);
        const uint16_t* pred = (const uint16_t*)(dlds + L.pred[k + 1]);
        const uint16_t* succ = (const uint16_t*)(dlds + L.succ[n - k]);
        const int cols_n = N[n - k - 1], cols_k = N[n - k];
        for (int e = tid; e < N[k + 1] * cols_n; e += kDenseBlock) {
            const int r = e / cols_n, q = e % cols_n;
            const double2* u = U + pred[2 * r * (k + 1)] * m;
            const float2* t = Tk + pred[2 * r * (k + 1) + 1] * cols_k;
            double2 acc = make_double2(0.0, 0.0);
            for (int i = 0; i < m; ++i) {
                const double2 a = u[i];
                const float2 v = t[succ[q * m + i]];
                acc.x = fma(a.x, (double)v.x, acc.x);
                acc.x = fma(-a.y, (double)v.y, acc.x);
                acc.y = fma(a.x, (double)v.y, acc.y);
                acc.y = fma(a.y, (double)v.x, acc.y);
            }
            Tn[e] = make_float2((float)acc.x, (float)acc.y);
        }
        __syncthreads();
    }
    const float* nrm = n > 0 ? ldc(&A.Ls[n].nrm) : nullptr;
    if constexpr (!BWD) {
        const float2* Tn = (const float2*)(dlds + L.T[n]);
        for (int t = tid; t < N[n]; t += kDenseBlock)
            A.y[o0 + t] = n > 0 ? c_scale(Tn[t], 1.f / ldg(nrm + t)) : Tn[t];
    } else {
        double2* gn = (double2*)(dlds + L.gn);
        const uint16_t* predn = (const uint16_t*)(dlds + L.pred[n]);
        for (int t = tid; t < N[n]; t += kDenseBlock) {
            const float2 v = A.gy[o0 + t];
            const double s = 1.0 / sqrt(fact_of(predn + 2 * t * n, n));
            gn[t] = make_double2(s * v.x, s * v.y);
        }
        __syncthreads();
        // thread (i, j, part): this part's share of gU[j][i]
        const int mm = m * m;
        const int parts = max(1, kDenseBlock / mm);
        double2 gu[(kMaxModes * kMaxModes + kDenseBlock - 1) / kDenseBlock];
#pragma unroll
        for (auto& v : gu) v = make_double2(0.0, 0.0);
        for (int k = n - 1; k >= 0; --k) {
            const float2* Tk = (const float2*)(dlds + L.T[k]);
            const double2* gu1 = (const double2*)(dlds + (k + 1 == n ? L.gn : L.g[(k + 1) & 1]));
            double2* gk = (double2*)(dlds + L.g[k & 1]);
            const uint16_t* succI = (const uint16_t*)(dlds + L.succ[n - k]);
            const uint16_t* succJ = (const uint16_t*)(dlds + L.succ[k + 1]);
            const uint16_t* predJ = (const uint16_t*)(dlds + L.pred[k + 1]);
            const uint16_t* predI = (const uint16_t*)(dlds + L.pred[n - k]);
            const uint16_t* firstJ = k > 0 ? (const uint16_t*)(dlds + L.pred[k]) : nullptr;
            const int32_t* minoff = ldc(&A.Ls[k + 1].minoff);
            const int cols_n = N[n - k - 1], cols_k = N[n - k];
#pragma unroll
            for (int w = 0; w < (int)(sizeof(gu) / sizeof(gu[0])); ++w) {
                const int e = tid + w * kDenseBlock, pr = e % mm, part = e / mm;
                if (part >= parts) break;
                const int j = pr / m, i = pr % m;
                const int lo = ldg(minoff + j), hi = ldg(minoff + j + 1);
                for (int r = lo; r < hi; ++r) {
                    const float2* t = Tk + predJ[2 * r * (k + 1) + 1] * cols_k;
                    for (int q = part; q < cols_n; q += parts) {
                        const float2 a = t[succI[q * m + i]];
                        z_fma_conj(gu[w], make_double2(a.x, a.y), gu1[r * cols_n + q]);
                    }
                }
            }
            for (int e = tid; e < N[k] * cols_k; e += kDenseBlock) {
                const int J = e / cols_k, I = e % cols_k;
                const int first = k > 0 ? firstJ[2 * J * k] : m - 1;
                double2 acc = make_double2(0.0, 0.0);
                for (int p = 0; p < n - k; ++p) {
                    const int i = predI[2 * (I * (n - k) + p)];
                    if (i == 0xFFFF) continue;
                    const double2* gq = gu1 + predI[2 * (I * (n - k) + p) + 1];
                    for (int j = 0; j <= first; ++j) z_fma_conj(acc, U[j * m + i], gq[succJ[J * m + j] * cols_n]);
                }
                gk[e] = acc;
            }
            __syncthreads();
        }
        if (A.gx) {
            const double2* g0 = (const double2*)(dlds + L.g[0]);
            for (int64_t c = c0 + tid; c < c1; c += kDenseBlock) {
                const int s = ldg(A.crank + c);
                const double f = sqrt(fact_of(predn + 2 * s * n, n));
                A.gx[c] = make_float2((float)(f * g0[s].x), (float)(f * g0[s].y));
            }
        }
        double2* part = (double2*)(dlds + L.part);
        if (parts > 1) {  // one pass: parts * mm <= kDenseBlock
            part[tid] = gu[0];
            __syncthreads();
            if (tid < mm) {
                double2 v = part[tid];
                for (int q = 1; q < parts; ++q) {
                    v.x += part[q * mm + tid].x;
                    v.y += part[q * mm + tid].y;
                }
                A.gU[(size_t)g * mm + tid] = (cols >> (tid % m)) & 1 ? make_float2((float)v.x, (float)v.y) : c_zero();
            }
        } else {
#pragma unroll
            for (int w = 0; w < (int)(sizeof(gu) / sizeof(gu[0])); ++w) {
                const int e = tid + w * kDenseBlock;
                if (e < mm) A.gU[(size_t)g * mm + e] = (cols >> (e % m)) & 1 ? make_float2((float)gu[w].x, (float)gu[w].y) : c_zero();
            }
        }
    }
}

size_t dense_lds(const slos_plan_s& P, int n, bool bwd) {
    int N[kMaxPhotons + 1];
    for (int k = 0; k <= n; ++k) N[k] = (int)P.N[k];
    DenseLayout L;
    dense_layout(N, P.m, n, bwd, L);
    return L.bytes;
}

}  // namespace

// Whether an input of `comps` distinct components of n photons can go through
// the steps above: they take no more products than one simulation per component
// (below that the component route is kept, as its results for a single component
// are those of the plain amplitudes bit for bit), and the adjoint fits in 80 KB of
// LDS (two workgroups a CU; most take half of that or less).
bool dense_superposition_ok(const slos_plan_s& P, int n, int64_t comps) {
    if (restricted_plan(P) || (P.flags & SLOS_PLAN_FORWARD_ONLY) || n < 1) return false;
    int64_t steps = 0, single = 0;
    for (int k = 1; k <= n; ++k) {
        if (P.N[k] > 4096 || P.N[k] * P.N[n - k] > 8192) return false;  // LDS, and 16-bit ranks
        steps += P.N[k] * P.N[n - k] * P.m;
        single += k * P.N[k];
    }
    return steps <= single * comps && dense_lds(P, n, true) <= 80 * 1024;
}

// Whether the steps are also sooner done.  They take one workgroup per input, so
// their time is that of one input's chain of steps until the inputs fill the chip
// twice over; one simulation per component spreads its components over the chip,
// and walks an input's components one after another only to combine them.  Both
// fitted, us, to measurements at 19 spaces (1 to 256 inputs, the fewest
// components and all of them): the adjoint's chain 4 + 4 n + (0.7 + 0.65 n) per 1000
// products, the forward's a 3.6th; one simulation per component 14 + 1.5 n + 0.055 m^2,
// 0.23 per component of an input and 0.022 or more per component beyond 512 (without
// dL/dx, as in training with fixed inputs), the forward 11, 0.52 and 0.006.  Either side
// of the line, steps / components: adjoint m = 8, n = 4, 17 of 330 states, 16 inputs 115
// / 35, 256 inputs 115 / 133, all states, 4 inputs 115 / 142; m = 6, n = 4, 11 of 126, 1
// input 45 / 30, all 45 / 59; m = 3, n = 8, all 45, 16 inputs 57 / 56, 64 inputs 56 / 133;
// m = 6, n = 3, all 56, 1 input 18 / 38; forward m = 6, n = 5, 13 of 252, 16 inputs 29 / 17,
// m = 8, n = 4, 41 of 330, 1 input 29 / 41.
bool dense_superposition_sooner(const slos_plan_s& P, int n, int64_t comps, int64_t inputs, int64_t all_comps,
                                bool bwd) {
    double steps = 0, single = 0;
    for (int k = 1; k <= n; ++k) {
        steps += (double)P.N[k] * P.N[n - k] * P.m;
        single += (double)k * P.N[k];
    }
    const double mm = (double)P.m * P.m, beyond = (double)std::max<int64_t>(0, all_comps - 512);
    const int64_t at_once = std::max(P.num_cu, 1) * (int64_t)(160 * 1024 / dense_lds(P, n, bwd));
    const double rounds = (double)((inputs + at_once - 1) / at_once);
    const double chain = (4.0 + 4.0 * n + steps * (0.7 + 0.65 * n) * 1e-3) * rounds;
    if (!bwd) return chain / 3.6 <= 11.0 + 0.52 * comps + 0.006 * beyond;
    const double each = std::max(0.022, std::max(0.012e-3 * single, 0.9e-4 * mm));
    return chain <= 14.0 + 1.5 * n + 0.055 * mm + 0.23 * comps + each * beyond;
}

int launch_dense_superposition(const SupDev& S, const slos_batch_s& Bt, bool bwd, const float2* U, const float2* x,
                               const float2* gy, float2* out, float2* gx, hipStream_t stream) {
    const slos_plan_s& P = *Bt.plan;
    DenseArgs A{P.m, P.d_layers, Bt.dev, S.goff, S.ooff, S.crank, S.cnorm, S.gcols, U, x, gy,
                bwd ? nullptr : out, bwd ? out : nullptr, gx};
    size_t lds = 0;
    for (int n = 1; n <= Bt.n_max; ++n)
        if (S.n_present >> n & 1) lds = std::max(lds, dense_lds(P, n, bwd));
    void* fn = bwd ? (void*)&dense_kernel<true> : (void*)&dense_kernel<false>;
    (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    void* args[] = {(void*)&A};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)S.G), dim3(kDenseBlock), args, lds, stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("dense superposition launch: ") + hipGetErrorString(e));
    return SLOS_OK;
}

}  // namespace slos
