// Fock spaces beyond on-chip memory by the two-halves evaluation
// (slos_halves.h): the halves' factors in the workspace, the outputs from them by
// matrix instructions.
//
// Layer by layer, every state of such a space is gathered from up to n states
// far apart in a layer larger than the caches (m = 24, n = 8, 16 samples: the last
// layer fetches 3.1 GB, a line at a time, for 0.5 GB of probabilities; 0.99 ms the
// forward).
// The halves' factors are 8.3 MB per half and sample, read in tiles; the cost is
// arithmetic instead, 47 complex products per output at the FP32 matrix rate.
// The same forward takes 0.81 ms: 0.57 ms of matrix products (25.5 million
// instructions, 0.40 ms at the measured 16 ns each per SIMD; vector
// instructions do not overlap with FP32 matrix ones on a SIMD), 0.04 ms the
// outputs with one photon in a half, 0.17 ms the factor tables.  Error of p
// against 64 bits 2.2e-7 by layers, 1.7e-7 here (level sums in FP64, products in
// chains of at most 32).
#include <type_traits>

#include "slos_halves.h"

namespace slos {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kBuildBlock = 256;
constexpr int64_t kHalvesMaxStates = (int64_t)1 << 27;  // output offsets below kNoByte
// Factor tables of one pass over the batch: few passes (m = 24, n = 8, 64 samples
// 3.07 ms at 512 MiB, 3.30 at 192, 4.20 at 48: each pass ends in a partly filled
// chip), and a workspace that does not grow with the batch.
constexpr size_t kHalvesWsBytes = (size_t)512 << 20;
constexpr uint32_t kNoByte = 0x60000000u;  // past every output buffer, also twice over: the access is dropped

__device__ __forceinline__ float2 ldg2(const float2* p) {
    typedef __attribute__((ext_vector_type(2))) float v2;
    const v2 v = *(__attribute__((address_space(1))) const v2*)p;
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ float2 buf_ld2(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, 0, 0));
}

// Level 1: the input photons' columns of U, [n][modes of the half].
__global__ __launch_bounds__(kBuildBlock) void halves_columns_kernel(HalvesDev H, BatchDev Bt, int m,
                                                                     const float2* __restrict__ U,
                                                                     float2* __restrict__ T) {
    const int b = blockIdx.x;
    for (int e = threadIdx.x; e < m * H.n; e += kBuildBlock) {
        const int j = e % m, i = e / m;
        const float2 v = U[((size_t)b * m + j) * m + ldg(Bt.modes + (size_t)b * kMaxPhotons + i)];
        const int s = j >= H.c;
        T[(size_t)b * H.per_sample + (s ? H.toff[1][1] : H.toff[0][1]) + i * H.mh[s] + (s ? j - H.c : j)] = v;
    }
}

// The parent row, first mode and weight of row r of level L of half s.
struct ChildRow {
    int j, parent;
    double f;
};
template <int L>
__device__ __forceinline__ ChildRow child_row(const HalvesDev& H, int s, int r, const int* mo) {
    // mo: LDS copy of the half's minoff rows, [level][kMaxModes + 1]
    constexpr int W = kMaxModes + 1;
    int lo = 0, hi = H.mh[s] - 1;  // the last j with minoff_L(j) <= r
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (mo[L * W + mid] <= r) lo = mid;
        else hi = mid - 1;
    }
    ChildRow c;
    c.j = lo;
    const int o = r - mo[L * W + lo];  // the parent's place among the states of level L-1 with first mode >= j
    c.parent = mo[(L - 1) * W + lo] + o;
    int mu = 1;  // the parents that begin with t copies of j come first, one for each state of level L-1-t from j on
#pragma unroll
    for (int t = 1; t < L; ++t) mu += o < (L - 1 - t > 0 ? H.D[s][L - 1 - t] - mo[(L - 1 - t) * W + lo] : 1);
    c.f = H.rs[mu];
    return c;
}

// Level L of both halves from level L-1, one row per thread; the tables are
// [subset][row], so loads and stores stream.  OUT 1, 2: level n as
// probabilities or amplitudes to the output (0: to the table).
template <int N, int L, int OUT>
__global__ __launch_bounds__(kBuildBlock) void halves_build_kernel(HalvesDev H, BatchDev Bt, float2* __restrict__ T,
                                                                   void* __restrict__ out) {
    constexpr int KP = sub_binom(N, L - 1), KC = sub_binom(N, L), W = kMaxModes + 1;
    __shared__ float2 u[kMaxModes * N];
    __shared__ int mo[(kHalvesMaxN + 1) * W];
    const int b = blockIdx.z, s = blockIdx.y, rows = H.D[s][L];
    if ((int)blockIdx.x * kBuildBlock >= rows) return;
    float2* Tb = T + (size_t)b * H.per_sample;
    const int mh = H.mh[s];
    for (int e = threadIdx.x; e < mh * N; e += kBuildBlock) u[(e % mh) * N + e / mh] = Tb[H.toff[s][1] + e];
    for (int e = threadIdx.x; e < (L + 1) * W; e += kBuildBlock)
        mo[e] = ldg(H.minoff + s * (kHalvesMaxN + 1) * W + e);
    __syncthreads();
    const int r = blockIdx.x * kBuildBlock + threadIdx.x;
    if (r >= rows) return;
    const ChildRow c = child_row<L>(H, s, r, mo);
    const float2* src = Tb + H.toff[s][L - 1] + c.parent;
    const int dp = H.D[s][L - 1];
    // the sums in FP64 (as fast as FP32 here), so that a level adds one rounding
    float2 v[KP];
    double2 uj[N];
#pragma unroll
    for (int q = 0; q < KP; ++q) v[q] = ldg2(src + (size_t)q * dp);
#pragma unroll
    for (int i = 0; i < N; ++i) uj[i] = make_double2(c.f * u[c.j * N + i].x, c.f * u[c.j * N + i].y);
    constexpr SubsetTerms<N, L> S;
#pragma unroll
    for (int q = 0; q < KC; ++q) {
        double2 z = make_double2(0.0, 0.0);
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const double2 a = uj[S.i[q][t]];
            const double x = v[S.src[q][t]].x, y = v[S.src[q][t]].y;
            z.x = fma(a.x, x, z.x);
            z.x = fma(-a.y, y, z.x);
            z.y = fma(a.x, y, z.y);
            z.y = fma(a.y, x, z.y);
        }
        const float2 w = make_float2((float)z.x, (float)z.y);
        if constexpr (OUT == 0) {
            Tb[H.toff[s][L] + (size_t)q * rows + r] = w;
        } else {
            const float in = ldc(Bt.innorm + b);
            const int64_t at = ldc(Bt.off + b) + (s == 0 ? ldg(H.base + H.boff[N] + r) : ldc(H.base + H.boff[0]) + r);
            const float2 a = c_scale(w, in);
            if (OUT == 1) ((float*)out)[at] = a.x * a.x + a.y * a.y;
            else ((float2*)out)[at] = a;
        }
    }
}

// ------------------------------------------------------------------ forward

// Tiles of kTA x kTB outputs (alpha, beta) of one (sample, k), four waves of
// 32 x 64 each, the inner length staged kChunk subsets at a time.  Rows of a
// staged chunk are padded so that two subsets' rows start 32 banks apart: an
// operand read of 16 rows of two subsets then covers all banks.
constexpr int kTA = 64, kTB = 128, kChunk = 16;
constexpr int kRA = 80, kRB = 144;
static_assert((2 * kRA) % 64 == 32 && (2 * kRB) % 64 == 32, "two subsets' rows start 32 banks apart");

__host__ __device__ __forceinline__ int halves_tiles(const HalvesDev& H, int k) {
    return (H.D[0][k] + kTA - 1) / kTA * ((H.D[1][H.n - k] + kTB - 1) / kTB);
}

// Element kk = 2 S + c of a row (c = 0 real, 1 imaginary): re += (A, -A)[kk] B[kk],
// im += A[kk ^ 1] B[kk], with B's subset S^c.  Each chunk's 32 products go into
// fresh accumulators, so that rounding grows with the chunk and not with the
// whole inner length (up to 140).
template <bool PROBS>
__global__ __launch_bounds__(256, 2) void halves_fwd_kernel(HalvesDev H, BatchDev Bt, const float2* __restrict__ T,
                                                            void* __restrict__ out, int ntiles) {
    __shared__ float2 As[2][kChunk * kRA];  // the chunk's A as (re, im), and as (-im, re) for the odd lane groups
    __shared__ float2 Bs[kChunk * kRB];
    const int b = blockIdx.x / ntiles, n = H.n;
    int k = 2, tile = blockIdx.x % ntiles;
    for (; k < n - 2; ++k) {
        const int t = halves_tiles(H, k);
        if (tile < t) break;
        tile -= t;
    }
    const int DA = H.D[0][k], DB = H.D[1][n - k];
    const int nb = (DB + kTB - 1) / kTB, a0 = tile / nb * kTA, b0 = tile % nb * kTB;
    int K = 1;
    for (int i = 1; i <= k; ++i) K = K * (n - i + 1) / i;
    const float2* Tb = T + (size_t)b * H.per_sample;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15, odd = g & 1;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = 32 * (wave >> 1), wb = 64 * (wave & 1);  // the wave's corner of the tile
    const float in = ldc(Bt.innorm + b);
    const int64_t off = ldc(Bt.off + b), len_out = ldc(Bt.off + b + 1) - off;
    constexpr uint32_t EB = PROBS ? 4u : 8u;
    const __amdgpu_buffer_rsrc_t ro = buf_rsrc((const char*)out + off * EB, (uint32_t)len_out * EB);
    // equal chunks of an even number of subsets
    const int nch = (K + kChunk - 1) / kChunk, len = ((K + nch - 1) / nch + 1) & ~1;
    constexpr int QA = kChunk * kTA / 256, QB = kChunk * kTB / 256;
    // (subsets past the last one lie outside the tables' buffers and read as zero)
    const __amdgpu_buffer_rsrc_t rA = buf_rsrc(Tb + H.toff[0][k], (uint32_t)(K * DA) * 8u);
    const __amdgpu_buffer_rsrc_t rB = buf_rsrc(Tb + H.toff[1][n - k], (uint32_t)(K * DB) * 8u);
    const __amdgpu_buffer_rsrc_t rbase = buf_rsrc(H.base + H.boff[k], (uint32_t)DA * 4u);
    const uint32_t vA = (uint32_t)((tid / kTA) * DA + min(a0 + tid % kTA, DA - 1)) * 8u;
    const uint32_t vB = (uint32_t)((K - 1 - tid / kTB) * DB + min(b0 + tid % kTB, DB - 1)) * 8u;
    float2 la[QA], lb[QB];
    auto fetch = [&](int S0) {
#pragma unroll
        for (int q = 0; q < QA; ++q) la[q] = buf_ld2(rA, vA + (uint32_t)((S0 + q * (256 / kTA)) * DA) * 8u);
#pragma unroll
        for (int q = 0; q < QB; ++q) lb[q] = buf_ld2(rB, vB - (uint32_t)((S0 + q * (256 / kTB)) * DB) * 8u);
    };
    const float2* pa = As[odd] + (g >> 1) * kRA + wa + c;
    const float* pb = (const float*)(Bs + (g >> 1) * kRB + wb + c) + odd;
    f4 re[2][4], im[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) re[i][j] = im[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    const bool idle = a0 + wa >= DA || b0 + wb >= DB;
    uint32_t row[2][4];
    fetch(0);
    for (int S0 = 0; S0 < K; S0 += len) {
        if (S0 > 0) __syncthreads();  // the last chunk has been read
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            const int e = (tid + q * 256) / kTA * kRA + (tid + q * 256) % kTA;
            As[0][e] = la[q];
            As[1][e] = make_float2(-la[q].y, la[q].x);
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) Bs[(tid + q * 256) / kTB * kRB + (tid + q * 256) % kTB] = lb[q];
        __syncthreads();
        const bool last = S0 + len >= K;
        if (!last) fetch(S0 + len);
        if (!idle) {
            if (last) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        row[i][q] = buf_ld1(rbase, (uint32_t)min(a0 + wa + 16 * i + 4 * g + q, DA - 1) * 4u, 0);
            }
            // every chunk takes the same number of steps (what is past the last
            // subset is zero), known when compiling: no branch between products
            auto multiply = [&](auto STEPS) {
                f4 cr[2][4], ci[2][4];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) cr[i][j] = ci[i][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < decltype(STEPS)::value; ++s) {
                    float2 av[2];
                    float bv[4];
#pragma unroll
                    for (int i = 0; i < 2; ++i) av[i] = pa[2 * s * kRA + 16 * i];
#pragma unroll
                    for (int j = 0; j < 4; ++j) bv[j] = pb[2 * (2 * s * kRB + 16 * j)];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            cr[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i].x, bv[j], cr[i][j], 0, 0, 0);
                            ci[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i].y, bv[j], ci[i][j], 0, 0, 0);
                        }
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        re[i][j] += cr[i][j];
                        im[i][j] += ci[i][j];
                    }
            };
            switch (len / 2) {  // inner lengths 15 to 70 in chunks of up to 16: 5 to 8 steps
                case 5: multiply(std::integral_constant<int, 5>{}); break;
                case 6: multiply(std::integral_constant<int, 6>{}); break;
                case 7: multiply(std::integral_constant<int, 7>{}); break;
                default: multiply(std::integral_constant<int, 8>{}); break;
            }
        }
    }
    if (idle) return;
    uint32_t col[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int y = b0 + wb + 16 * j + c;
        col[j] = y < DB ? (uint32_t)y * EB : kNoByte;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t r = a0 + wa + 16 * i + 4 * g + q < DA ? row[i][q] * EB : kNoByte;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float ar = in * re[i][j][q], ai = in * im[i][j][q];
                if (PROBS) {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ar * ar + ai * ai), ro, (int)(r + col[j]), 0, 0);
                } else {
                    typedef __attribute__((ext_vector_type(2))) unsigned int u2;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, make_float2(ar, ai)), ro,
                                                          (int)(r + col[j]), 0, 0);
                }
            }
        }
}

// One photon in a half (s = 0: k = 1, s = 1: k = n-1): n products per output, too
// few for a tile.  A thread takes a row of the other half's level n-1 (its n
// factors in registers, loads coalesced) and the few modes of this half.
template <int N, bool PROBS>
__global__ __launch_bounds__(kBuildBlock) void halves_edge_kernel(HalvesDev H, BatchDev Bt, const float2* __restrict__ T,
                                                                  void* __restrict__ out) {
    __shared__ float2 u[kMaxModes * N];  // this half's columns, [mode][photon]
    __shared__ int first[kMaxModes];     // s = 0: rank of (mode, first beta)
    const int b = blockIdx.z, s = blockIdx.y, rows = H.D[1 - s][N - 1], mh = H.mh[s];
    if ((int)blockIdx.x * kBuildBlock >= rows) return;
    const float2* Tb = T + (size_t)b * H.per_sample;
    for (int e = threadIdx.x; e < mh * N; e += kBuildBlock) u[e % mh * N + e / mh] = Tb[H.toff[s][1] + e];
    if (s == 0 && (int)threadIdx.x < mh) first[threadIdx.x] = ldg(H.base + H.boff[1] + threadIdx.x);
    __syncthreads();
    const int r = blockIdx.x * kBuildBlock + threadIdx.x;
    if (r >= rows) return;
    const float2* src = Tb + H.toff[1 - s][N - 1] + r;
    float2 v[N];  // v[i]: the other half without photon i, subset N-1-i of level N-1
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = ldg2(src + (size_t)(N - 1 - i) * rows);
    const float in = ldc(Bt.innorm + b);
    const int64_t off = ldc(Bt.off + b);
    const int64_t own = s == 0 ? r : ldg(H.base + H.boff[N - 1] + r);
    for (int j = 0; j < mh; ++j) {
        float2 w = c_zero();
#pragma unroll
        for (int i = 0; i < N; ++i) c_fma(w, u[j * N + i], v[i]);
        w = c_scale(w, in);
        const int64_t at = off + own + (s == 0 ? first[j] : j);
        if (PROBS) ((float*)out)[at] = w.x * w.x + w.y * w.y;
        else ((float2*)out)[at] = w;
    }
}

template <int N, int L>
int halves_levels(const HalvesDev& H, const BatchDev& dev, int nb, float2* T, void* out, bool probs,
                  hipStream_t stream) {
    if constexpr (L <= N) {
        const int rows = std::max(H.D[0][L], H.D[1][L]);
        void* fn = L < N   ? (void*)&halves_build_kernel<N, L, 0>
                   : probs ? (void*)&halves_build_kernel<N, N, 1>
                           : (void*)&halves_build_kernel<N, N, 2>;
        void* args[] = {(void*)&H, (void*)&dev, (void*)&T, (void*)&out};
        hipError_t e = hipLaunchKernel(fn, dim3((unsigned)((rows + kBuildBlock - 1) / kBuildBlock), 2, (unsigned)nb),
                                       dim3(kBuildBlock), args, 0, stream);
        if (e != hipSuccess) return fail(SLOS_EHIP, std::string("two-halves level launch: ") + hipGetErrorString(e));
        return halves_levels<N, L + 1>(H, dev, nb, T, out, probs, stream);
    } else {
        return SLOS_OK;
    }
}

// Levels 1 .. n-1 of both halves into T, level n to the output.
int halves_tables(const HalvesDev& H, const BatchDev& dev, int nb, int m, const float2* U, float2* T, void* out,
                  bool probs, hipStream_t stream) {
    void* args[] = {(void*)&H, (void*)&dev, (void*)&m, (void*)&U, (void*)&T};
    hipError_t e = hipLaunchKernel((void*)&halves_columns_kernel, dim3((unsigned)nb), dim3(kBuildBlock), args, 0, stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("two-halves launch: ") + hipGetErrorString(e));
    switch (H.n) {
        case 6: return halves_levels<6, 2>(H, dev, nb, T, out, probs, stream);
        case 7: return halves_levels<7, 2>(H, dev, nb, T, out, probs, stream);
        default: return halves_levels<8, 2>(H, dev, nb, T, out, probs, stream);
    }
}

int halves_ntiles(const HalvesDev& H) {
    int t = 0;
    for (int k = 2; k < H.n - 1; ++k) t += halves_tiles(H, k);
    return t;
}

}  // namespace

// Every sample the same photon number, in a space whose tables the plan holds.
bool halves_served(const slos_batch_s& Bt) {
    if (Bt.B < 1 || Bt.n_min != Bt.n_max || Bt.n_max > kHalvesMaxN) return false;
    return Bt.plan->halves[Bt.n_max].n != 0 && Bt.plan->N[Bt.n_max] <= kHalvesMaxStates;
}

// A space large enough that layers miss the caches, and outputs enough to pay for
// the n + 2 launches and their tables: 5 million states, which is every space of 8
// photons that has tables (the plan builds none below), or 16 (n = 7) and 8 (n = 6)
// million outputs.  Both sides measured, us, layer by layer against two halves.  n = 8: m = 22 (4.3
// million states) 4 samples 167 / 166, m = 23 (5.9) 1 sample 104 / 91, m = 24
// (7.9) 1 sample 135 / 101, 16 samples 995 / 812, m = 28 (23.5) 1 sample 340 / 184.  n = 7:
// m = 20 (0.66) 32 samples 152 / 159, m = 24 (2.0) 8 samples 118 / 121, m = 26 (3.4)
// 2 samples 69 / 75, 5 samples 192 / 121, m = 28 (5.4) 1 sample 83 / 64.  n = 6: m = 24
// (0.48) 16 samples 70 / 66, m = 28 (1.1) 4 samples 49 / 48, 8 samples 69 / 65, 32
// samples 207 / 159.  n = 5 gains 10 % at most (m = 32, 32 samples 81 / 73) and is
// left to the layers.
bool halves_ok(const slos_batch_s& Bt) {
    if (!halves_served(Bt)) return false;
    const int64_t N = Bt.plan->N[Bt.n_max];
    return N >= 5000000 || (Bt.n_max < 8 && N * Bt.B >= (Bt.n_max == 6 ? 8000000 : 16000000));
}

// Samples per pass: equal passes whose factor tables stay below kHalvesWsBytes.
int halves_pass(const slos_batch_s& Bt) {
    const size_t all = (size_t)Bt.B * Bt.plan->halves[Bt.n_max].per_sample * sizeof(float2);
    const int passes = (int)std::min<size_t>((all + kHalvesWsBytes - 1) / kHalvesWsBytes, Bt.B);
    return (Bt.B + passes - 1) / passes;
}

size_t halves_ws_bytes(const slos_batch_s& Bt) {
    return (size_t)halves_pass(Bt) * Bt.plan->halves[Bt.n_max].per_sample * sizeof(float2);
}

int launch_halves_fwd(const slos_batch_s& Bt, const float2* U, void* out, bool probs, void* ws, hipStream_t stream) {
    const HalvesDev& H = Bt.plan->halves[Bt.n_max];
    float2* T = (float2*)ws;
    const int pass = halves_pass(Bt), m = Bt.plan->m;
    const int rows = std::max(H.D[0][H.n - 1], H.D[1][H.n - 1]);
    int ntiles = halves_ntiles(H);
    void* edge = H.n == 6   ? (probs ? (void*)&halves_edge_kernel<6, true> : (void*)&halves_edge_kernel<6, false>)
                 : H.n == 7 ? (probs ? (void*)&halves_edge_kernel<7, true> : (void*)&halves_edge_kernel<7, false>)
                            : (probs ? (void*)&halves_edge_kernel<8, true> : (void*)&halves_edge_kernel<8, false>);
    void* tile = probs ? (void*)&halves_fwd_kernel<true> : (void*)&halves_fwd_kernel<false>;
    for (int b0 = 0; b0 < Bt.B; b0 += pass) {
        const int nb = std::min(pass, Bt.B - b0);
        BatchDev dev = Bt.dev;  // the pass's samples; outputs stay where off puts them
        dev.modes += (size_t)b0 * kMaxPhotons;
        dev.off += b0;
        dev.innorm += b0;
        int rc = halves_tables(H, dev, nb, m, U + (size_t)b0 * m * m, T, out, probs, stream);
        if (rc != SLOS_OK) return rc;
        void* eargs[] = {(void*)&H, (void*)&dev, (void*)&T, (void*)&out};
        hipError_t e = hipLaunchKernel(edge, dim3((unsigned)((rows + kBuildBlock - 1) / kBuildBlock), 2, (unsigned)nb),
                                       dim3(kBuildBlock), eargs, 0, stream);
        void* args[] = {(void*)&H, (void*)&dev, (void*)&T, (void*)&out, (void*)&ntiles};
        if (e == hipSuccess) e = hipLaunchKernel(tile, dim3((unsigned)(nb * ntiles)), dim3(256), args, 0, stream);
        if (e != hipSuccess) return fail(SLOS_EHIP, std::string("two-halves forward launch: ") + hipGetErrorString(e));
    }
    return SLOS_OK;
}

}  // namespace slos
