// Layered kernels: one launch per photon layer, with the layers kept in the
// caller's workspace instead of LDS.  They handle Fock spaces of any size
// (a photon layer may be far larger than a workgroup's LDS) and, with
// B = 1, serve as the unbatched per-sample path.
//
// Same recursion as the fused kernels (arXiv 2602.11092, Sec. II-A-3):
// layer k is pulled from layer k-1 through the transition tables.  The
// batch is split into groups of SG samples (SG a power of two <= 8) and
// each layer is stored [group][state][SG], so the lanes that share a
// state read one contiguous SG*8-byte segment per gather.  The backward
// recomputes layers 1..n-1 into the workspace, then walks k = n..1 with a
// seed launch (top-layer gradient of the samples whose top is layer k), a
// pull launch (g_{k-1} and the partial sums of G_U[:, i_k]) and, at the
// end, one launch that adds the partial sums in a fixed order.
//
// Bound by the gathers past the L2s: of a state's k neighbours the ones that
// differ in an early photon are far away.  What that costs depends on how much
// is in flight and how long a line stays, hence: lanes of two samples (16-byte
// loads; half the addresses, table entries and instructions), a state's gathers
// issued together with the next state's table entries behind them, groups of
// 8 samples (64-byte segments; with 64 samples a group the same window of states
// is eight times the bytes), one contiguous eighth of the states per XCD, and a
// grid that is resident at once.  Forward and adjoint, us, before -> now: m = 24,
// n = 8, 16 samples 1502 -> 995, 2766 -> 2140; m = 20, n = 6, 64 samples 265 -> 85, 469 ->
// 203; m = 14, n = 7, 64 samples 152 -> 68, 306 -> 160; m = 24, n = 8, 1 sample 145 -> 135,
// 469 -> 333.  The top layers at m = 24, n = 8, 16 samples: the seed fetches 3.6 GB (5.9
// before) and writes 1.0 in 0.97 ms, the first pull 4.1 (5.4) and 0.26 in 0.73 ms: 4.8
// and 6.0 TB/s, a large copy's rate; neither more wavefronts nor earlier loads help
// any further.
#include "slos_internal.h"

namespace slos {
namespace {

// Blocks of a pull launch along the states, over all groups about two grids of
// four per CU (its registers allow 4 waves per SIMD): m = 24, n = 8, 16 samples
// 2175 us with 1024, 2327 with 768 and 2339 with 2048.  A layer launch keeps about 5
// per CU: m = 20, n = 6, 512 samples 1321 us with 2560 over all groups, 1643 with 2048
// for each group; a layer that 2560 blocks cover is given all it needs (m = 28,
// n = 5, 2 samples 21 us in 1280).
constexpr int kPullBlocks = 1024, kLayerBlocks = 2560;
// Values (states x samples) of a layer from which its lanes take two samples:
// smaller ones do not fill the chip and run on more wavefronts (forward, us: m = 12,
// n = 8, 3 samples 34 with pairs throughout, 28.5 now; m = 16, n = 7, 1 sample 25 and
// 23; m = 20, n = 6, 3 samples 24.9, 23.9 and 25.4 from 2^16, 2^19 and 2^20 values).
constexpr int64_t kPairLanes = 1 << 19;
// The lanes of a state share its successors, a part of the modes each: 2 parts for
// lanes of two samples (4: m = 24, n = 8, 16 samples 2398 us against 2175), 4 for a
// lone sample (1, 2, 4, 8 parts: 624, 370, 333, 361 us).
constexpr int kParts1 = 4, kParts2 = 2;

struct Shape {
    int SG;    // samples per group (lanes sharing a state)
    int NGRP;  // number of groups
    int GX;    // blocks along the state axis in the pull launches
};

// Groups of 8 samples: m = 20, n = 6, 64 samples 272 us with 8, 277 with 16, 344
// with 64, 294 with 4; m = 28, n = 5, 40 samples 222, 241, 316, 250.  (64 for batches whose
// groups of 8 would not fit the grid.)
Shape shape_of(const slos_batch_s& Bt) {
    const int most = Bt.B <= 8 * 32768 ? 8 : 64;
    int sg = 1;
    while (sg < Bt.B && sg < most) sg <<= 1;
    const int ngrp = (Bt.B + sg - 1) / sg;
    // no more blocks than the largest pull range needs (256 threads each)
    const int64_t Nmax = Bt.n_max >= 1 ? Bt.plan->N[Bt.n_max - 1] : 1;
    const int64_t need = (Nmax * sg + 255) / 256 * (sg > 1 ? 1 : kParts1);
    const int cap = std::max(8, std::min(kPullBlocks, 2 * kPullBlocks / ngrp));
    int gx = (int)std::max<int64_t>(1, std::min<int64_t>(need, cap));
    if (gx >= 64) gx = (gx + 7) & ~7;
    return Shape{sg, ngrp, gx};
}

// Blocks of a pull over Nprev states: no more than have work.
__host__ __device__ __forceinline__ int pull_blocks(int64_t Nprev, int SG, int GX) {
    const int64_t need = (Nprev * (SG > 1 ? SG / 2 * kParts2 : kParts1) + 255) / 256;
    const int gx = need < GX ? (int)need : GX;
    return gx >= 64 ? (gx + 7) & ~7 : gx;  // (GX, too, is a multiple of 8 from 64 on)
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace layout.
struct Layout {
    size_t store_off[kMaxPhotons + 1];  // bwd: layer k at store_off[k] (k = 1..n_max-1)
    size_t buf0, buf1;                  // fwd: ping-pong layers; bwd: g ping-pong
    size_t partial;                     // bwd: [n_max][NGRP][GX][SG][32] float2
    size_t col;                         // bwd: [B][kMaxPhotons][32] float2, G_U[:, i_k] per layer
    size_t total;
};

Layout layout_of(const slos_batch_s& Bt, bool backward) {
    const slos_plan_s& P = *Bt.plan;
    const Shape sh = shape_of(Bt);
    const size_t per_state = (size_t)sh.NGRP * sh.SG * sizeof(float2);
    Layout L{};
    size_t off = 0;
    int64_t maxN = 1;
    if (backward) {
        for (int k = 1; k <= Bt.n_max - 1; ++k) {
            L.store_off[k] = off;
            off += align256((size_t)P.N[k] * per_state);
        }
        for (int k = 1; k <= Bt.n_max; ++k) maxN = std::max(maxN, P.N[k]);
    } else {
        for (int k = 1; k <= Bt.n_max - 1; ++k) maxN = std::max(maxN, P.N[k]);
    }
    L.buf0 = off;
    off += align256((size_t)maxN * per_state);
    L.buf1 = off;
    off += align256((size_t)maxN * per_state);
    L.partial = off;
    if (backward) off += align256((size_t)std::max(Bt.n_max, 1) * sh.NGRP * sh.GX * sh.SG * 32 * sizeof(float2));
    L.col = off;
    if (backward) off += align256((size_t)Bt.B * kMaxPhotons * 32 * sizeof(float2));
    L.total = off;
    return L;
}

// A block's states of [0, N): workgroups are dealt to the eight XCDs in turn, so
// with a grid of a multiple of eight each XCD is given one contiguous eighth.
struct Range {
    int t, end, step;
};
__device__ __forceinline__ Range block_range(int N, int TPB, int tl) {
    const int xcds = gridDim.x % 8 == 0 ? 8 : 1;
    const int seg = (N + xcds - 1) / xcds, lo = (int)(blockIdx.x % xcds) * seg;
    return Range{lo + (int)(blockIdx.x / xcds) * TPB + tl, min(N, lo + seg), (int)(gridDim.x / xcds) * TPB};
}


enum Mode { kForward = 0, kRecompute = 1, kSeed = 2 };

// V adjacent samples of one state.
template <int V>
struct Vec {
    float2 s[V];
};
template <int V>
__device__ __forceinline__ Vec<V> ld_vec(const float2* p) {
    Vec<V> r;
    if constexpr (V == 2) {
        const float4 v = *(const float4*)p;
        r.s[0] = make_float2(v.x, v.y);
        r.s[1] = make_float2(v.z, v.w);
    } else {
        r.s[0] = *p;
    }
    return r;
}

template <int V>
__device__ __forceinline__ void st_vec(float2* p, const Vec<V>& x, const bool (&on)[V], bool all) {
    if (V == 2 && all) {
        *(float4*)p = make_float4(x.s[0].x, x.s[0].y, x.s[V - 1].x, x.s[V - 1].y);
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (on[v]) p[v] = x.s[v];
    }
}

// One layer for every active sample of a group.  kForward: samples whose top
// layer is k write their outputs, the others write layer k.  kRecompute:
// only samples with more than k photons, writing layer k.  kSeed: only
// samples whose top layer is k, writing g_k.  A lane takes V samples (2 when the
// group has as many), one 16-byte load each for the state and the coefficient.
template <int BLOCK, bool PROBS, int V>
__global__ __launch_bounds__(BLOCK) void layered_layer_kernel(int m, const LayerDev* __restrict__ Ls, BatchDev Bt,
                                                              const float2* __restrict__ U, int k, int mode,
                                                              const float2* __restrict__ prev, float2* __restrict__ cur,
                                                              void* __restrict__ out, const void* __restrict__ gin,
                                                              int SG) {
    __shared__ __attribute__((aligned(16))) float2 us[64 * kUcolSlots];  // [slot][SG]
    const int tid = threadIdx.x;
    const int per = SG / V;  // lanes of one state
    const int bl = tid % per * V;
    const int tl = tid / per;
    const int TPB = BLOCK / per;
    const int g = blockIdx.y;
    // what the first state needs besides the column is on its way while the
    // column is staged
    const int N = (int)ldc(&Ls[k].N), Nprev = (int)ldc(&Ls[k - 1].N);
    const int sh = ldc(&Ls[k].pred_shift), ngrp = ldc(&Ls[k].ngrp);
    const uint4* predv = ldc(&Ls[k].predv);
    const float* nrms = ldc(&Ls[k].nrm);
    const uint32_t rmask = pred_rank_mask(sh);
    const bool need_d = !(mode == kSeed && !PROBS), table = need_d && k > 1;
    const Range R = block_range(N, TPB, tl);
    uint4 e0 = {}, e1 = {};
    if (table && R.t < R.end) {
        e0 = predv[R.t];
        if (ngrp > 1) e1 = predv[(size_t)N + R.t];
    }
    int n_b[V];
    float innorm[V];
    int64_t off[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int b = min(g * SG + bl + v, Bt.B - 1);
        n_b[v] = Bt.n[b];
        innorm[v] = Bt.innorm[b];
        off[v] = Bt.off[b];
    }
    // stage column i_k of U for every sample of the group (slot 32 = 0)
    for (int q = tid; q < SG; q += BLOCK) us[32 * SG + q] = c_zero();
    for (int q = tid; q < SG * m; q += BLOCK) {
        const int bq = q % SG, j = q / SG;
        const int bb = g * SG + bq;
        if (bb < Bt.B && Bt.n[bb] >= k) {
            const int ik = Bt.modes[(size_t)bb * kMaxPhotons + k - 1];
            us[j * SG + bq] = U[((size_t)bb * m + j) * m + ik];
        }
    }
    __syncthreads();
    bool active[V], top[V], any = false, all = true;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const bool here = g * SG + bl + v < Bt.B;
        active[v] = here && (mode == kForward ? n_b[v] >= k : mode == kRecompute ? n_b[v] > k : n_b[v] == k);
        top[v] = n_b[v] == k;
        any |= active[v];
        all &= active[v];
    }
    if (!any) return;
    const float2* pg = prev + (size_t)g * Nprev * SG + bl;
    for (int t = R.t; t < R.end; t += R.step) {
        // (the state's norm and incoming gradient fly with its gathers)
        const float nrm = mode == kRecompute ? 0.f : nrms[t];
        Vec<V> acc;
        float2 gi[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            acc.s[v] = gi[v] = c_zero();
            if (mode != kSeed || !active[v]) continue;
            if (PROBS) gi[v].x = ((const float*)gin)[off[v] + t];
            else gi[v] = ((const float2*)gin)[off[v] + t];
        }
        if (table) {
            // two groups' gathers in flight at once, and the next state's entries behind them
            const uint4 c0 = e0, c1 = e1;
            const uint32_t es[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
            Vec<V> d[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) d[q] = ld_vec<V>(pg + (size_t)((es[q] & rmask) >> 3) * SG);
            if (ngrp > 1) {
#pragma unroll
                for (int q = 4; q < 8; ++q) d[q] = ld_vec<V>(pg + (size_t)((es[q] & rmask) >> 3) * SG);
            }
            if (t + R.step < R.end) {
                e0 = predv[t + R.step];
                if (ngrp > 1) e1 = predv[(size_t)N + t + R.step];
            }
            // empty entries name the zero slot 32 of the coefficient column
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const Vec<V> u = ld_vec<V>(us + (es[q] >> sh) * SG + bl);
#pragma unroll
                for (int v = 0; v < V; ++v) c_fma(acc.s[v], u.s[v], d[q].s[v]);
            }
            if (ngrp > 1) {
#pragma unroll
                for (int q = 4; q < 8; ++q) {
                    const Vec<V> u = ld_vec<V>(us + (es[q] >> sh) * SG + bl);
#pragma unroll
                    for (int v = 0; v < V; ++v) c_fma(acc.s[v], u.s[v], d[q].s[v]);
                }
            }
            for (int gq = 2; gq < ngrp; ++gq) {
                const uint4 e4 = predv[(size_t)gq * N + t];
                const uint32_t ex[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const Vec<V> u = ld_vec<V>(us + (ex[q] >> sh) * SG + bl);
                    const Vec<V> x = ld_vec<V>(pg + (size_t)((ex[q] & rmask) >> 3) * SG);
#pragma unroll
                    for (int v = 0; v < V; ++v) c_fma(acc.s[v], u.s[v], x.s[v]);
                }
            }
        } else if (need_d) {
            acc = ld_vec<V>(us + t * SG + bl);
        }
        float2* to = cur + ((size_t)g * N + t) * SG + bl;
        bool store[V], both = all;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            store[v] = active[v];
            if (!active[v]) continue;
            if (mode == kForward && top[v]) {
                const float c = nrm * innorm[v];
                const float2 a = acc.s[v];
                if (PROBS) ((float*)out)[off[v] + t] = c * c * (a.x * a.x + a.y * a.y);
                else ((float2*)out)[off[v] + t] = c_scale(a, c);
                store[v] = both = false;
            } else if (mode == kSeed) {
                const float c = nrm * innorm[v];
                if (PROBS) acc.s[v] = c_scale(acc.s[v], 2.f * gi[v].x * c * c);
                else acc.s[v] = c_scale(gi[v], c);
            }
        }
        st_vec<V>(to, acc, store, both);
    }
}

// g_{k-1}[t'] = sum_j conj(u_j) g_k[t'+e_j]; partial sums of
// G_U[j][i_k] = sum_t' conj(d_{k-1}[t']) g_k[t'+e_j] per block.  A lane takes V
// samples and one of PARTS shares of the modes (MMAX in all), whose G_U partials
// it keeps in registers (modes past m read padding successors and zero
// coefficients and are never written out); the lanes of a state add their
// shares of g_{k-1} across the wave, and the block adds the lanes of each
// sample in a fixed order through LDS, four modes at a time.
// RESTRICTED: plans of a restricted space, whose successor tables mark
// successors outside the space with kNoSuccessor; those pairs contribute
// nothing (the forward never formed such states).
template <int BLOCK, int MMAX, bool RESTRICTED, int V, int PARTS>
__global__ __launch_bounds__(BLOCK) void layered_pull_kernel(int m, const LayerDev* __restrict__ Ls, BatchDev Bt,
                                                             const float2* __restrict__ U, int k,
                                                             const float2* __restrict__ gk, float2* __restrict__ gkm1,
                                                             const float2* __restrict__ dkm1,
                                                             float2* __restrict__ partial, int SG, int NGRP, int GX) {
    constexpr int G = (MMAX / 4 + PARTS - 1) / PARTS;  // successor groups (of four modes) per lane
    __shared__ __attribute__((aligned(16))) float2 lds[64 * kUcolSlots];
    static_assert(4 * V * BLOCK <= 64 * kUcolSlots, "the lanes' sums reuse the column's memory");
    float2* us = lds;  // [slot][SG]
    const int tid = threadIdx.x;
    const int per = SG / V, lanes = per * PARTS;  // lanes of one state
    const int bl = tid % per * V, part = tid / per % PARTS;  // samples bl .. bl+V-1, modes from 4 G part on
    const int tl = tid / lanes;
    const int TPB = BLOCK / lanes;
    const int g = blockIdx.y;
    bool active[V], any = false, all = true;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int b = g * SG + bl + v;
        active[v] = b < Bt.B && Bt.n[b] >= k;
        any |= active[v];
        all &= active[v];
    }
    for (int q = tid; q < SG * kUcolSlots; q += BLOCK) us[q] = c_zero();
    __syncthreads();
    for (int q = tid; q < SG * m; q += BLOCK) {
        const int bq = q % SG, j = q / SG;
        const int bb = g * SG + bq;
        if (bb < Bt.B && Bt.n[bb] >= k) {
            const int ik = Bt.modes[(size_t)bb * kMaxPhotons + k - 1];
            us[j * SG + bq] = U[((size_t)bb * m + j) * m + ik];
        }
    }
    __syncthreads();
    Vec<V> h[4 * G];
#pragma unroll
    for (int j = 0; j < 4 * G; ++j)
#pragma unroll
        for (int v = 0; v < V; ++v) h[j].s[v] = c_zero();
    if (any) {
        const int Nk = (int)Ls[k].N;
        const int Nkm1 = (int)Ls[k - 1].N;
        const int ngs = (m + 3) >> 2;  // successor groups in the table
        const uint4* succ4 = (const uint4*)Ls[k].succ + (size_t)min(G * part, ngs - 1) * Nkm1;
        const int mine = ngs - G * part;  // this lane's groups
        const float2* gkg = gk + (size_t)g * Nk * SG + bl;
        const float2* ul = us + 4 * G * part * SG + bl;
        const Range R = block_range(Nkm1, TPB, tl);
        for (int tp = R.t; tp < R.end; tp += R.step) {
            Vec<V> dv, acc;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                dv.s[v] = make_float2(1.f, 0.f);
                acc.s[v] = c_zero();
            }
            if (k >= 2) dv = ld_vec<V>(dkm1 + ((size_t)g * Nkm1 + tp) * SG + bl);
            uint4 s4[G];
#pragma unroll
            for (int q4 = 0; q4 < G; ++q4) s4[q4] = succ4[(size_t)(q4 < mine ? q4 : 0) * Nkm1 + tp];
#pragma unroll
            for (int q4 = 0; q4 < G; ++q4) {
                if (q4 >= mine) continue;
                const uint32_t sv[4] = {s4[q4].x, s4[q4].y, s4[q4].z, s4[q4].w};
                Vec<V> gv[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool none = RESTRICTED && sv[q] == kNoSuccessor;
                    gv[q] = ld_vec<V>(gkg + (size_t)((none ? 0u : sv[q]) >> 3) * SG);
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (none) gv[q].s[v] = c_zero();
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const Vec<V> u = ld_vec<V>(ul + (4 * q4 + q) * SG);
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        c_fma_conj(acc.s[v], u.s[v], gv[q].s[v]);
                        c_fma_conj(h[4 * q4 + q].s[v], dv.s[v], gv[q].s[v]);
                    }
                }
            }
            if (k >= 2) {
                float2* to = gkm1 + ((size_t)g * Nkm1 + tp) * SG + bl;
#pragma unroll
                for (int x = 1; x < PARTS; x *= 2)
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        acc.s[v].x += __shfl_xor(acc.s[v].x, x * per);
                        acc.s[v].y += __shfl_xor(acc.s[v].y, x * per);
                    }
                if (part == 0) st_vec<V>(to, acc, active, all);
            }
        }
    }
    // fixed-order sum over the lanes that share a sample, one group at a time
#pragma unroll
    for (int q4 = 0; q4 < G; ++q4) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int v = 0; v < V; ++v) lds[(V * q + v) * BLOCK + tid] = h[4 * q4 + q].s[v];
        __syncthreads();
        for (int e = tid; e < SG * PARTS * 4; e += BLOCK) {
            const int s = e % SG, pt = e / SG % PARTS, q = e / SG / PARTS;
            const int j = 4 * (G * pt + q4) + q;
            if (j >= 32) continue;
            const float2* src = lds + (V * q + s % V) * BLOCK + pt * per + s / V;
            float2 sum = c_zero();
            for (int tq = 0; tq < TPB; ++tq) sum = c_add(sum, src[tq * lanes]);
            partial[((((size_t)(k - 1) * NGRP + g) * GX + blockIdx.x) * SG + s) * 32 + j] = sum;
        }
    }
}

// Column i_k of G_U for sample b from layer k's block partials.  One block
// per (sample, layer): 32 slices of 32 lanes (one lane per mode) each add
// every 32nd block partial with eight independent accumulators, then the
// slices are added in order.  The order is fixed, so results are
// reproducible; the loads of a slice are all independent.
__global__ __launch_bounds__(1024) void layered_reduce_kernel(const LayerDev* __restrict__ Ls, BatchDev Bt,
                                                              const float2* __restrict__ partial,
                                                              float2* __restrict__ col, int SG, int NGRP, int GX) {
    __shared__ float2 part[32][33];
    const int b = blockIdx.x;
    const int k = blockIdx.y + 1;
    if (k > Bt.n[b]) return;  // uniform over the block
    const int g = b / SG, bl = b % SG;
    const int tid = threadIdx.x, j = tid & 31, sl = tid >> 5;
    const float2* src = partial + (((size_t)(k - 1) * NGRP + g) * GX * SG + bl) * 32 + j;
    const size_t xs = (size_t)SG * 32;  // stride between consecutive block partials
    float2 a[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = c_zero();
    const int nx = pull_blocks(Ls[k - 1].N, SG, GX);
    int x = sl;
    for (; x + 7 * 32 < nx; x += 8 * 32) {
#pragma unroll
        for (int q = 0; q < 8; ++q) a[q] = c_add(a[q], src[(size_t)(x + q * 32) * xs]);
    }
    for (; x < nx; x += 32) a[0] = c_add(a[0], src[(size_t)x * xs]);
    float2 v = c_zero();
#pragma unroll
    for (int q = 0; q < 8; ++q) v = c_add(v, a[q]);
    part[sl][j] = v;
    __syncthreads();
    if (tid < 32) {
        float2 sum = c_zero();
        for (int q = 0; q < 32; ++q) sum = c_add(sum, part[q][tid]);
        col[((size_t)b * kMaxPhotons + k - 1) * 32 + tid] = sum;
    }
}

// G_U[b][j][i] = sum over photon layers k with i_k = i of column k, in k order.
__global__ __launch_bounds__(256) void layered_final_kernel(int m, BatchDev Bt, const float2* __restrict__ col,
                                                            float2* __restrict__ gU) {
    const int b = blockIdx.x;
    const int n_b = Bt.n[b];
    const int32_t* modes = Bt.modes + (size_t)b * kMaxPhotons;
    const float2* cb = col + (size_t)b * kMaxPhotons * 32;
    for (int q = threadIdx.x; q < m * m; q += blockDim.x) {
        const int jj = q / m, i = q % m;
        float2 v = c_zero();
        for (int k = 1; k <= n_b; ++k)
            if (modes[k - 1] == i) v = c_add(v, cb[(k - 1) * 32 + jj]);
        gU[(size_t)b * m * m + q] = v;
    }
}

// Samples without photons: the only output is the vacuum, amplitude 1.
__global__ void vacuum_kernel(BatchDev Bt, void* out, int probs) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= Bt.B || Bt.n[b] != 0) return;
    if (probs) ((float*)out)[Bt.off[b]] = 1.f;
    else ((float2*)out)[Bt.off[b]] = make_float2(1.f, 0.f);
}

template <bool PROBS, int V>
void* layer_fn(int block) {
    switch (block) {
        case 64: return (void*)&layered_layer_kernel<64, PROBS, V>;
        case 128: return (void*)&layered_layer_kernel<128, PROBS, V>;
        case 256: return (void*)&layered_layer_kernel<256, PROBS, V>;
        case 512: return (void*)&layered_layer_kernel<512, PROBS, V>;
        case 1024: return (void*)&layered_layer_kernel<1024, PROBS, V>;
    }
    return nullptr;
}

int launch_layer(const slos_batch_s& Bt, int block, const float2* U, int k, int mode, const float2* prev,
                 float2* cur, void* out, const void* gin, bool probs, hipStream_t stream) {
    const slos_plan_s& P = *Bt.plan;
    const Shape sh = shape_of(Bt);
    if (block < sh.SG) block = sh.SG;
    const int V = sh.SG > 1 && P.N[k] * sh.SG * sh.NGRP >= kPairLanes ? 2 : 1;
    void* fn = V == 2 ? (probs ? layer_fn<true, 2>(block) : layer_fn<false, 2>(block))
                      : (probs ? layer_fn<true, 1>(block) : layer_fn<false, 1>(block));
    if (!fn) return fail(SLOS_EUNSUPPORTED, "layered: bad block size");
    const int TPB = block / (sh.SG / V);
    const int64_t N = P.N[k];
    const int64_t need = (N + TPB - 1) / TPB;
    int gx = (int)(need * sh.NGRP <= kLayerBlocks ? need : std::max(8, std::min(kLayerBlocks / 2, kLayerBlocks / sh.NGRP)));
    if (gx >= 64) gx = (gx + 7) & ~7;
    int m = P.m;
    const LayerDev* Ls = P.d_layers;
    int SG = sh.SG;
    void* args[] = {(void*)&m, (void*)&Ls, (void*)&Bt.dev, (void*)&U, (void*)&k, (void*)&mode,
                    (void*)&prev, (void*)&cur, (void*)&out, (void*)&gin, (void*)&SG};
    hipError_t e = hipLaunchKernel(fn, dim3(gx, sh.NGRP), dim3(block), args, 0, stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("layered layer launch: ") + hipGetErrorString(e));
    return SLOS_OK;
}

}  // namespace

size_t layered_ws_bytes(const slos_batch_s& Bt, bool backward) {
    if (Bt.B == 0 || Bt.n_max == 0) return 0;
    return layout_of(Bt, backward).total;
}

int layered_default_block(const slos_batch_s& Bt) {
    (void)Bt;
    return 256;
}

int launch_layered_fwd(const slos_batch_s& Bt, int block, const float2* U, void* out, bool probs, void* ws,
                       hipStream_t stream) {
    const Layout L = layout_of(Bt, false);
    char* base = (char*)ws;
    float2* bufs[2] = {(float2*)(base + L.buf0), (float2*)(base + L.buf1)};
    for (int k = 1; k <= Bt.n_max; ++k) {
        const float2* prev = bufs[(k - 1) & 1];
        float2* cur = bufs[k & 1];
        int rc = launch_layer(Bt, block, U, k, kForward, prev, cur, out, nullptr, probs, stream);
        if (rc != SLOS_OK) return rc;
    }
    bool any_vacuum = false;
    for (int b = 0; b < Bt.B; ++b) any_vacuum |= (Bt.n_host[b] == 0);
    if (any_vacuum) {
        int pr = probs ? 1 : 0;
        void* args[] = {(void*)&Bt.dev, (void*)&out, (void*)&pr};
        hipError_t e = hipLaunchKernel((void*)&vacuum_kernel, dim3((Bt.B + 255) / 256), dim3(256), args, 0, stream);
        if (e != hipSuccess) return fail(SLOS_EHIP, std::string("vacuum launch: ") + hipGetErrorString(e));
    }
    return SLOS_OK;
}

template <bool R, int V, int PARTS>
static void* pull_fn_r(int m) {
    if (m <= 8) return (void*)&layered_pull_kernel<256, 8, R, V, PARTS>;
    if (m <= 12) return (void*)&layered_pull_kernel<256, 12, R, V, PARTS>;
    if (m <= 16) return (void*)&layered_pull_kernel<256, 16, R, V, PARTS>;
    if (m <= 20) return (void*)&layered_pull_kernel<256, 20, R, V, PARTS>;
    if (m <= 24) return (void*)&layered_pull_kernel<256, 24, R, V, PARTS>;
    return (void*)&layered_pull_kernel<256, 32, R, V, PARTS>;
}

static void* pull_fn(int m, bool restricted, int V) {
    if (V == 2) return restricted ? pull_fn_r<true, 2, kParts2>(m) : pull_fn_r<false, 2, kParts2>(m);
    return restricted ? pull_fn_r<true, 1, kParts1>(m) : pull_fn_r<false, 1, kParts1>(m);
}

int launch_layered_bwd(const slos_batch_s& Bt, int block, const float2* U, const void* gin, bool probs, float2* gU,
                       void* ws, hipStream_t stream) {
    const slos_plan_s& P = *Bt.plan;
    const Shape sh = shape_of(Bt);
    const Layout L = layout_of(Bt, true);
    char* base = (char*)ws;
    auto store = [&](int k) -> float2* { return (k >= 1) ? (float2*)(base + L.store_off[k]) : nullptr; };
    float2* gbuf[2] = {(float2*)(base + L.buf0), (float2*)(base + L.buf1)};
    float2* partial = (float2*)(base + L.partial);
    int rc;
    for (int k = 1; k <= Bt.n_max - 1; ++k) {
        rc = launch_layer(Bt, block, U, k, kRecompute, store(k - 1), store(k), nullptr, nullptr, probs, stream);
        if (rc != SLOS_OK) return rc;
    }
    int m = P.m;
    const LayerDev* Ls = P.d_layers;
    int SG = sh.SG, NGRP = sh.NGRP, GX = sh.GX;
    for (int k = Bt.n_max; k >= 1; --k) {
        float2* gk = gbuf[(Bt.n_max - k) & 1];
        float2* gkm1 = gbuf[(Bt.n_max - k + 1) & 1];
        // the seed writes g_k of the samples whose top layer is k; with none, g_k
        // is the previous pull's output as it stands
        bool any_top = false;
        for (int b = 0; b < Bt.B && !any_top; ++b) any_top = (Bt.n_host[b] == k);
        if (any_top) {
            rc = launch_layer(Bt, block, U, k, kSeed, store(k - 1), gk, nullptr, gin, probs, stream);
            if (rc != SLOS_OK) return rc;
        }
        const float2* dkm1 = store(k - 1);
        void* args[] = {(void*)&m, (void*)&Ls, (void*)&Bt.dev, (void*)&U, (void*)&k, (void*)&gk,
                        (void*)&gkm1, (void*)&dkm1, (void*)&partial, (void*)&SG, (void*)&NGRP, (void*)&GX};
        const bool restricted = (P.flags & (SLOS_PLAN_UNBUNCHED | SLOS_PLAN_DUAL_RAIL)) != 0;
        hipError_t e = hipLaunchKernel(pull_fn(m, restricted, SG > 1 ? 2 : 1), dim3(pull_blocks(P.N[k - 1], SG, GX), NGRP), dim3(256), args, 0, stream);
        if (e != hipSuccess) return fail(SLOS_EHIP, std::string("layered pull launch: ") + hipGetErrorString(e));
    }
    float2* col = (float2*)(base + L.col);
    {
        void* args[] = {(void*)&Ls, (void*)&Bt.dev, (void*)&partial, (void*)&col, (void*)&SG, (void*)&NGRP, (void*)&GX};
        hipError_t e = hipLaunchKernel((void*)&layered_reduce_kernel, dim3(Bt.B, std::max(Bt.n_max, 1)), dim3(1024), args, 0, stream);
        if (e != hipSuccess) return fail(SLOS_EHIP, std::string("layered reduce launch: ") + hipGetErrorString(e));
    }
    void* args[] = {(void*)&m, (void*)&Bt.dev, (void*)&col, (void*)&gU};
    hipError_t e = hipLaunchKernel((void*)&layered_final_kernel, dim3(Bt.B), dim3(256), args, 0, stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("layered final launch: ") + hipGetErrorString(e));
    return SLOS_OK;
}

}  // namespace slos
