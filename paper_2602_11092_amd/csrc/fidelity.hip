// Fidelity kernel between output states of one input Fock state under two
// interferometers (the kernel-methods reproduction of Sec. III-A):
//
//   K[a][b] = |<phi(U1_a)|phi(U2_b)>|^2,   |phi(U)> = U|s>,
//   <phi(U1)|phi(U2)> = Perm(M) / prod_i s_i!,   M = U1[:, C]^H U2[:, C],
//
// where C lists the input modes with multiplicity (n x n; Cauchy-Binet over
// the output basis turns the inner product of two C(m+n-1, n)-dimensional
// vectors into one n x n permanent).  FP64 arithmetic on the complex64 inputs
// (the chip's FP64 vector rate equals its unpacked FP32 rate, and the
// permanent's sums of signed products cancel strongly).
//
// Three kernels:
//  * n <= 8: a workgroup takes a 16 x 16 tile of (a, b) pairs (8 x 8 at n = 8) and
//    stages the input columns of its 32 (16) unitaries in LDS (a thread's own loads
//    of them are strided by a whole unitary: 64 cache lines an instruction, which is
//    what the time went into).  Perm(M) by Glynn's formula over column signs,
//      Perm(M) = 2^(1-n) sum_{delta, delta_0 = 1} prod_j delta_j prod_i sum_j delta_j M[i][j],
//    half of Ryser's terms, in Gray-code order and unrolled for the
//    compile-time n, so every index into M is static.  Up to n = 7 a thread
//    owns a pair, M in registers (n = 7: 224 of 256 VGPRs).  At n = 8 four
//    lanes share a pair: each forms two columns of M, passed through LDS, and
//    sums the 32 terms of its signs of columns 1 and 2.
//    A Gram matrix (U1 = U2) is symmetric: only tiles on and above the
//    diagonal are formed, and mirrored.
//    Bound by the FP64 vector rate: M takes 4 n^2 m products a pair, the sum
//    2^(n-1) (6 n - 2).  us before (a thread per pair, Ryser, no staging; n = 8
//    a wave per pair) and now, Gram matrices: m = 6, n = 4, B = 1024 56 / 22;
//    m = 20, n = 5, B = 512 82 / 28; m = 10, n = 7, B = 512 94 / 52; m = 12, n = 8,
//    B = 512 846 / 116.  n = 6 and 7 on four lanes too: 30 -> 44 and 52 -> 55 (LDS
//    reads); n = 8 on two: 116 -> 190.
//  * n = 3 to 7, K of a few long rows or columns: a thread per pair (the rule and
//    both sides' times stand at fid_few_rows).
//  * n >= 9 (and n = 0, and a single row at n = 8): one wave per pair.  Its lanes build M in LDS, then
//    lane l walks the Gray-code positions [l K, (l+1) K), K = ceil(2^n / 64),
//    of Ryser's formula,
//      Perm(M) = (-1)^n sum_{S subset of [n]} (-1)^|S| prod_i sum_{j in S} M[i][j],
//    from row sums formed directly, one column added or removed per step; a
//    fixed-order shuffle reduction combines the lanes.
#include "slos_internal.h"

namespace slos {
namespace {

constexpr int kFidBlock = 256;
constexpr int kFidWaves = kFidBlock / 64;
constexpr int kFidMaxN = kMaxPhotons;

struct FidModes {
    int32_t c[kFidMaxN];  // input modes with multiplicity, ascending
};

__device__ __forceinline__ double2 z_mul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Pairs per side of a tile.
constexpr int fid_tile(int q) { return q == 0 ? 16 : 8; }

// Product of the row sums, factors in pairs: half the chain of dependent FP64
// products.
template <int N>
__device__ __forceinline__ double2 z_prod(const double2 (&rs)[N]) {
    if constexpr (N == 1) {
        return rs[0];
    } else {
        double2 prod = z_mul(rs[0], rs[1]);
#pragma unroll
        for (int i = 2; i + 1 < N; i += 2) prod = z_mul(prod, z_mul(rs[i], rs[i + 1]));
        if (N % 2 == 1) prod = z_mul(prod, rs[N - 1]);
        return prod;
    }
}

// Glynn's sum over the signs of F columns, M2 twice the columns: sum of
// prod_j delta_j prod_i rs_i, rs the row sums with every delta_j = 1.  Leaves rs
// at the last step's signs: column F-1 negated.
template <int N, int F>
__device__ __forceinline__ double2 glynn_sum(double2 (&rs)[N], const double2 (&M2)[F > 0 ? F : 1][N]) {
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < (1 << F); ++q) {
        if (q > 0) {  // one column changes its sign
            const int j = __builtin_ctz(q);
            const bool neg = ((q ^ (q >> 1)) >> j) & 1;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                rs[i].x = neg ? rs[i].x - M2[j][i].x : rs[i].x + M2[j][i].x;
                rs[i].y = neg ? rs[i].y - M2[j][i].y : rs[i].y + M2[j][i].y;
            }
        }
        const double2 prod = z_prod<N>(rs);
        if (__builtin_popcount(q ^ (q >> 1)) & 1) {
            acc.x -= prod.x;
            acc.y -= prod.y;
        } else {
            acc.x += prod.x;
            acc.y += prod.y;
        }
        // steps interleaved by the scheduler would not fit the registers
        asm volatile("" : "+v"(acc.x), "+v"(acc.y));
#pragma unroll
        for (int i = 0; i < N; ++i) asm volatile("" : "+v"(rs[i].x), "+v"(rs[i].y));
    }
    return acc;
}

// Q: 2^Q lanes share a pair (columns 1 .. Q have a sign per lane).
template <int N, int Q>
__global__ __launch_bounds__(fid_tile(Q) * fid_tile(Q) << Q) void fidelity_tile_kernel(
    int m, FidModes C, double scale, const float2* __restrict__ U1, int B1, const float2* __restrict__ U2, int B2,
    float* __restrict__ K, int tb, unsigned tiles, bool gram, bool cols) {
    constexpr int T = fid_tile(Q), LANES = 1 << Q, THREADS = T * T * LANES;
    const unsigned tile = blockIdx.y * gridDim.x + blockIdx.x;
    const int ty = (int)(tile / (unsigned)tb), tx = (int)(tile % (unsigned)tb);
    if (tile >= tiles || (gram && tx < ty)) return;
    // [2][m][N][T] columns of the tile's U1 and U2, widened once, then M of each pair (Q > 0)
    extern __shared__ double2 fid_lds[];
    const int tid = threadIdx.x;
    const int a0 = ty * T, b0 = tx * T;
    // a thread takes the N entries of a row of one unitary: N loads in flight
    for (int e = tid; e < 2 * T * m; e += THREADS) {
        const int x = e % T, row = e / T;  // row: k of U1, then of U2
        const bool second = row >= m;
        const int u = (second ? b0 : a0) + x, k = second ? row - m : row;
        const float2* src = (second ? U2 : U1) + (int64_t)min(u, (second ? B2 : B1) - 1) * m * m + k * m;
        float2 v[N];
#pragma unroll
        for (int c = 0; c < N; ++c) v[c] = src[C.c[c]];
#pragma unroll
        for (int c = 0; c < N; ++c) fid_lds[(row * N + c) * T + x] = make_double2(v[c].x, v[c].y);
    }
    __syncthreads();
    // Up to n = 7 a wave's pairs are four rows a by 16 columns b (cols, for K of few
    // columns: the other way round), so that where K ends inside a tile whole waves
    // have no pairs and stop: one row of 131072 at m = 10, n = 4 31 us (67 when the
    // rows past the last were computed too).
    const int pr = tid / LANES, part = tid % LANES;
    const int xa = Q == 0 && cols ? pr % T : pr / T, xb = Q == 0 && cols ? pr / T : pr % T;
    if constexpr (Q == 0) {
        const int first = __builtin_amdgcn_readfirstlane(pr / T);
        if (cols ? b0 + first >= B2 : a0 + first >= B1) return;
    }
    const double2* s1 = fid_lds + xa;
    const double2* s2 = fid_lds + T * m * N + xb;
    // columns NC part .. of M: M[r][c] = sum_k conj(U1[a][k][C_r]) U2[b][k][C_c]
    constexpr int NC = (N + LANES - 1) / LANES;  // (the last lane's may run past the last column)
    double2 M[NC][N];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < N; ++r) M[c][r] = make_double2(0.0, 0.0);
#pragma unroll 1
    for (int k = 0; k < m; ++k) {
        double2 x[N], y[NC];
#pragma unroll
        for (int r = 0; r < N; ++r) x[r] = s1[(k * N + r) * T];
#pragma unroll
        for (int c = 0; c < NC; ++c) y[c] = s2[(k * N + min(NC * part + c, N - 1)) * T];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int r = 0; r < N; ++r) {
                M[c][r].x = fma(x[r].x, y[c].x, M[c][r].x);
                M[c][r].x = fma(x[r].y, y[c].y, M[c][r].x);
                M[c][r].y = fma(x[r].x, y[c].y, M[c][r].y);
                M[c][r].y = fma(-x[r].y, y[c].x, M[c][r].y);
            }
    }
    double2 sum;
    if constexpr (Q == 0) {
        double2 rs[N], V[N > 1 ? N - 1 : 1][N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            rs[i] = M[0][i];
#pragma unroll
            for (int c = 1; c < N; ++c) {
                rs[i].x += M[c][i].x;
                rs[i].y += M[c][i].y;
                V[c - 1][i] = make_double2(M[c][i].x + M[c][i].x, M[c][i].y + M[c][i].y);
            }
        }
        sum = glynn_sum<N, N - 1>(rs, V);
    } else {
        // M of every pair through LDS, [column][row][pair]; the last three columns
        // in registers, eight steps each time one of those before them (columns
        // Q+1 ..) changes its sign
        double2* Ms = fid_lds + 2 * T * m * N;
        constexpr int P = T * T, REG = 3, OUTER = N - 1 - Q - REG;
        static_assert(OUTER >= 0, "the lanes and the registers hold at most the columns after the first");
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int r = 0; r < N; ++r)
                if (NC * part + c < N) Ms[((NC * part + c) * N + r) * P + pr] = M[c][r];
        __syncthreads();
        const double2* Mp = Ms + pr;
        double2 rs[N], V[REG][N];
#pragma unroll
        for (int i = 0; i < N; ++i) rs[i] = Mp[i * P];
#pragma unroll 1
        for (int c = 1; c < N - REG; ++c) {
            const double sg = c <= Q && ((part >> (c - 1)) & 1) ? -1.0 : 1.0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double2 v = Mp[(c * N + i) * P];
                rs[i].x = fma(sg, v.x, rs[i].x);
                rs[i].y = fma(sg, v.y, rs[i].y);
            }
        }
#pragma unroll
        for (int c = 0; c < REG; ++c)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double2 v = Mp[((N - REG + c) * N + i) * P];
                rs[i].x += v.x;
                rs[i].y += v.y;
                V[c][i] = make_double2(v.x + v.x, v.y + v.y);
            }
        sum = make_double2(0.0, 0.0);
#pragma unroll 1
        for (int q = 0; q < (1 << OUTER); ++q) {
            const int gray = q ^ (q >> 1);
            if (q > 0) {  // the outer column's sign, and the last register column's back
                const int j = __builtin_ctz(q);
                const double two = ((gray >> j) & 1) ? -2.0 : 2.0;
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const double2 v = Mp[((Q + 1 + j) * N + i) * P];
                    rs[i].x = fma(two, v.x, rs[i].x + V[REG - 1][i].x);
                    rs[i].y = fma(two, v.y, rs[i].y + V[REG - 1][i].y);
                }
            }
            const double sg = (__builtin_popcount(gray) & 1) ? -1.0 : 1.0;
            const double2 part8 = glynn_sum<N, REG>(rs, V);
            sum.x = fma(sg, part8.x, sum.x);
            sum.y = fma(sg, part8.y, sum.y);
        }
        if (__builtin_popcount(part) & 1) sum = make_double2(-sum.x, -sum.y);
#pragma unroll
        for (int s = 1; s < LANES; s <<= 1) {
            sum.x += __shfl_xor(sum.x, s, 64);
            sum.y += __shfl_xor(sum.y, s, 64);
        }
    }
    const int a = a0 + xa, b = b0 + xb;
    if (a >= B1 || b >= B2 || part != 0) return;
    constexpr double half = 1.0 / (1 << (N - 1));
    const double re = sum.x * half * scale, im = sum.y * half * scale;
    const float v = (float)(re * re + im * im);
    if (gram && a > b) return;  // the diagonal tile's lower half is mirrored too
    K[(int64_t)a * B2 + b] = v;
    if (gram && a < b) K[(int64_t)b * B2 + a] = v;
}

// A thread per pair, its columns read from memory (lanes of a wave share a):
// Ryser's formula over the subsets in Gray-code order, from the empty set.
template <int N>
__global__ __launch_bounds__(kFidBlock) void fidelity_thread_kernel(int m, FidModes C, double scale,
                                                                    const float2* __restrict__ U1, int B1,
                                                                    const float2* __restrict__ U2, int B2,
                                                                    float* __restrict__ K) {
    const int64_t pair = (int64_t)blockIdx.x * kFidBlock + threadIdx.x;
    if (pair >= (int64_t)B1 * B2) return;
    const int64_t a = pair / B2, b = pair % B2;
    const float2* u1 = U1 + a * m * m;
    const float2* u2 = U2 + b * m * m;
    // M[r][c] = sum_k conj(U1[a][k][C_r]) U2[b][k][C_c]
    double2 M[N][N];
#pragma unroll
    for (int r = 0; r < N; ++r)
#pragma unroll
        for (int c = 0; c < N; ++c) M[r][c] = make_double2(0.0, 0.0);
    for (int k = 0; k < m; ++k) {
        double2 x[N], y[N];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const float2 v = u1[k * m + C.c[r]], w = u2[k * m + C.c[r]];
            x[r] = make_double2(v.x, v.y);
            y[r] = make_double2(w.x, w.y);
        }
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int c = 0; c < N; ++c) {
                M[r][c].x += x[r].x * y[c].x + x[r].y * y[c].y;
                M[r][c].y += x[r].x * y[c].y - x[r].y * y[c].x;
            }
    }
    // Ryser over the subsets in Gray-code order, starting from the empty set
    double2 rs[N];
#pragma unroll
    for (int i = 0; i < N; ++i) rs[i] = make_double2(0.0, 0.0);
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 1; q < (1 << N); ++q) {
        const int j = __builtin_ctz(q);
        const int g = q ^ (q >> 1);
        const double sgn = ((g >> j) & 1) ? 1.0 : -1.0;  // column j enters or leaves
#pragma unroll
        for (int i = 0; i < N; ++i) {
            rs[i].x += sgn * M[i][j].x;
            rs[i].y += sgn * M[i][j].y;
        }
        double2 prod = rs[0];
#pragma unroll
        for (int i = 1; i < N; ++i) prod = z_mul(prod, rs[i]);
        const double sg = (__builtin_popcount(g) & 1) ? -1.0 : 1.0;
        acc.x += sg * prod.x;
        acc.y += sg * prod.y;
    }
    const double sn = (N & 1) ? -1.0 : 1.0;
    const double re = sn * acc.x * scale, im = sn * acc.y * scale;
    K[pair] = (float)(re * re + im * im);
}

// Whether K has too few rows (or columns) for tiles: a tile's waves take four of
// them, and once the tiles (one per 16 along the other side) fill the chip that
// work counts.  us, tiles / a thread per pair (n = 8: a wave per pair): n = 7, m = 10
// 32768 long 1 row 92 / 26, 4 rows 92 / 51, 6 rows 93 / 73, 8 rows 93 / 94, 4096 long
// 1 row 13 / 21; n = 6, m = 12 131072 long 1 row 81 / 45, 2 rows 83 / 81, 3 rows 86 / 114;
// n = 5, m = 20 32768 long 1 row 33 / 24, 2 rows 33 / 25, 3 rows 34 / 55, 131072 long
// (420 MB of unitaries, beyond the caches and read once per row) 2 rows 114 / 194;
// n = 4, m = 10 131072 long 1 row 32 / 25, 2 rows 32 / 52; n = 3, m = 6 1 row 13 / 11;
// n = 8, m = 12 32768 long 1 row 139 / 114, 2 rows 140 / 213.
bool fid_few_rows(int m, int n, int rows, int64_t length) {
    if (n == 8) return rows == 1;
    if (n == 7) return rows <= 6 && length > 4096;
    if (n < 3 || length <= 16384) return false;
    return rows == 1 || (rows == 2 && n >= 5 && length * m * m * (int64_t)sizeof(float2) <= ((int64_t)256 << 20));
}

__global__ __launch_bounds__(kFidBlock) void fidelity_kernel(int m, int n, FidModes C, double scale,
                                                             const float2* __restrict__ U1, int B1,
                                                             const float2* __restrict__ U2, int B2,
                                                             float* __restrict__ K) {
    __shared__ double2 Ms[kFidWaves][kFidMaxN * kFidMaxN];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t npairs = (int64_t)B1 * B2;
    const int T = 1 << n;                       // subsets
    const int chunk = (T + 63) / 64;            // Gray-code positions per lane
    // uniform trip count over the workgroup (the barriers below need it)
    for (int64_t base = (int64_t)blockIdx.x * kFidWaves; base < npairs; base += (int64_t)gridDim.x * kFidWaves) {
        const int64_t pair = base + w;
        const bool active = pair < npairs;
        const int64_t a = active ? pair / B2 : 0, b = active ? pair % B2 : 0;
        // M[r][c] = sum_k conj(U1[a][k][C_r]) U2[b][k][C_c]
        if (active) {
            const float2* u1 = U1 + a * m * m;
            const float2* u2 = U2 + b * m * m;
            for (int e = lane; e < n * n; e += 64) {
                const int r = e / n, c = e % n;
                const int cr = C.c[r], cc = C.c[c];
                double re = 0.0, im = 0.0;
                for (int k = 0; k < m; ++k) {
                    const float2 x = u1[k * m + cr], y = u2[k * m + cc];
                    re += (double)x.x * y.x + (double)x.y * y.y;
                    im += (double)x.x * y.y - (double)x.y * y.x;
                }
                Ms[w][e] = make_double2(re, im);
            }
        }
        __syncthreads();
        double2 acc = make_double2(0.0, 0.0);
        if (active) {
            const double2* M = Ms[w];
            const int q0 = lane * chunk, q1 = min(q0 + chunk, T);
            if (q0 < q1) {
                // row sums of the subset at Gray position q0
                const int g0 = q0 ^ (q0 >> 1);
                double2 rs[kFidMaxN];
#pragma unroll
                for (int i = 0; i < kFidMaxN; ++i) {
                    rs[i] = make_double2(0.0, 0.0);
                    if (i < n)
                        for (int j = 0; j < n; ++j)
                            if ((g0 >> j) & 1) {
                                rs[i].x += M[i * n + j].x;
                                rs[i].y += M[i * n + j].y;
                            }
                }
                int g = g0;
                for (int q = q0; q < q1; ++q) {
                    if (q > q0) {  // step to position q: one column enters or leaves
                        const int j = __builtin_ctz(q);
                        const double sgn = ((g >> j) & 1) ? -1.0 : 1.0;
                        g ^= 1 << j;
#pragma unroll
                        for (int i = 0; i < kFidMaxN; ++i)
                            if (i < n) {
                                rs[i].x += sgn * M[i * n + j].x;
                                rs[i].y += sgn * M[i * n + j].y;
                            }
                    }
                    double2 prod = make_double2(1.0, 0.0);
#pragma unroll
                    for (int i = 0; i < kFidMaxN; ++i)
                        if (i < n) prod = z_mul(prod, rs[i]);
                    const double sg = (__builtin_popcount(g) & 1) ? -1.0 : 1.0;
                    acc.x += sg * prod.x;
                    acc.y += sg * prod.y;
                }
            }
        }
        // fixed-order butterfly over the wave
        for (int s = 32; s >= 1; s >>= 1) {
            acc.x += __shfl_xor(acc.x, s, 64);
            acc.y += __shfl_xor(acc.y, s, 64);
        }
        if (active && lane == 0) {
            const double sn = (n & 1) ? -1.0 : 1.0;
            const double re = sn * acc.x * scale, im = sn * acc.y * scale;
            K[pair] = (float)(re * re + im * im);
        }
        __syncthreads();  // before the next pair overwrites Ms
    }
}

}  // namespace
}  // namespace slos

using namespace slos;

extern "C" int fock_fidelity_kernel(int m, const int32_t* occ, const float* U1, int B1, const float* U2, int B2,
                                    float* K, void* stream) {
    if (m < 1 || m > kMaxModes) return fail(SLOS_EINVAL, "fock_fidelity_kernel: m must be in [1, 32]");
    if (!occ) return fail(SLOS_EINVAL, "fock_fidelity_kernel: occ is NULL");
    if (B1 < 0 || B2 < 0) return fail(SLOS_EINVAL, "fock_fidelity_kernel: negative batch size");
    FidModes C{};
    int n = 0;
    double fact = 1.0;
    for (int i = 0; i < m; ++i) {
        if (occ[i] < 0) return fail(SLOS_EINVAL, "fock_fidelity_kernel: negative occupation");
        for (int q = 0; q < occ[i]; ++q) {
            if (n == kFidMaxN) return fail(SLOS_EUNSUPPORTED, "fock_fidelity_kernel: more than 16 photons");
            C.c[n++] = i;
            fact *= (q + 1);
        }
    }
    if ((int64_t)B1 * B2 == 0) return SLOS_OK;
    if (!U1 || !U2 || !K) return fail(SLOS_EINVAL, "fock_fidelity_kernel: NULL device pointer");
    const double scale = 1.0 / fact;
    const int q = n == 8 ? 2 : 0, T = fid_tile(q);
    const int64_t ta = ((int64_t)B1 + T - 1) / T, tb64 = ((int64_t)B2 + T - 1) / T;
    if (n >= 1 && n <= 7 && ta * tb64 >= ((int64_t)1 << 31))
        return fail(SLOS_EUNSUPPORTED, "fock_fidelity_kernel: too many pairs");
    const int64_t pair_blocks = ((int64_t)B1 * B2 + kFidBlock - 1) / kFidBlock;
    // (a dimension of a launch holds less than 2^32 threads)
    const bool few = fid_few_rows(m, n, std::min(B1, B2), std::max(B1, B2)) &&
                     (n == 8 || pair_blocks * kFidBlock < ((int64_t)1 << 32));
    if (few && n <= 7) {
        static void* const thread_fns[5] = {(void*)&fidelity_thread_kernel<3>, (void*)&fidelity_thread_kernel<4>,
                                            (void*)&fidelity_thread_kernel<5>, (void*)&fidelity_thread_kernel<6>,
                                            (void*)&fidelity_thread_kernel<7>};
        void* args[] = {(void*)&m, (void*)&C, (void*)&scale, (void*)&U1, (void*)&B1, (void*)&U2, (void*)&B2, (void*)&K};
        hipError_t e = hipLaunchKernel(thread_fns[n - 3], dim3((unsigned)pair_blocks), dim3(kFidBlock), args, 0,
                                       (hipStream_t)stream);
        if (e != hipSuccess)
            return fail(SLOS_EHIP, std::string("fock_fidelity_kernel launch: ") + hipGetErrorString(e));
        return SLOS_OK;
    }
    if (n >= 1 && n <= 8 && !few && ta * tb64 < ((int64_t)1 << 31)) {
        static void* const tile_fns[8] = {(void*)&fidelity_tile_kernel<1, 0>, (void*)&fidelity_tile_kernel<2, 0>,
                                          (void*)&fidelity_tile_kernel<3, 0>, (void*)&fidelity_tile_kernel<4, 0>,
                                          (void*)&fidelity_tile_kernel<5, 0>, (void*)&fidelity_tile_kernel<6, 0>,
                                          (void*)&fidelity_tile_kernel<7, 0>, (void*)&fidelity_tile_kernel<8, 2>};
        const size_t lds = (size_t)2 * T * m * n * sizeof(double2) + (q > 0 ? (size_t)n * n * T * T * sizeof(double2) : 0);
        int tb = (int)tb64;
        unsigned tiles = (unsigned)(ta * tb64);
        const unsigned gx = std::min(tiles, 1u << 23), gy = (tiles + gx - 1) / gx;
        bool gram = U1 == U2 && B1 == B2, cols = B2 < B1 && B2 < T;
        void* fn = tile_fns[n - 1];
        (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        void* args[] = {(void*)&m, (void*)&C, (void*)&scale, (void*)&U1, (void*)&B1, (void*)&U2, (void*)&B2, (void*)&K,
                        (void*)&tb, (void*)&tiles, (void*)&gram, (void*)&cols};
        hipError_t e = hipLaunchKernel(fn, dim3(gx, gy), dim3(T * T << q), args, lds, (hipStream_t)stream);
        if (e != hipSuccess)
            return fail(SLOS_EHIP, std::string("fock_fidelity_kernel launch: ") + hipGetErrorString(e));
        return SLOS_OK;
    }
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(SLOS_EHIP, "fock_fidelity_kernel: no HIP device");
    hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t blocks = ((int64_t)B1 * B2 + kFidWaves - 1) / kFidWaves;
    const int grid = (int)std::min<int64_t>(blocks, (int64_t)std::max(cu, 1) * 8);
    void* args[] = {(void*)&m, (void*)&n, (void*)&C, (void*)&scale, (void*)&U1, (void*)&B1,
                    (void*)&U2, (void*)&B2, (void*)&K};
    hipError_t e = hipLaunchKernel((void*)&fidelity_kernel, dim3(grid), dim3(kFidBlock), args, 0,
                                   (hipStream_t)stream);
    if (e != hipSuccess) return fail(SLOS_EHIP, std::string("fock_fidelity_kernel launch: ") + hipGetErrorString(e));
    return SLOS_OK;
}
