// k_als.hip -- CP-ALS on the GPU (Sec. 2.3, eqs. cp_nls and cp_als), FP64: the
// right-hand sides of the three least-squares subproblems (matricized tensor times
// Khatri-Rao product, as an FP64 MFMA product with one factor followed by an elementwise
// reduction with the other) and their normal matrices (elementwise products of factor
// Grams).  The normal equations are solved by the SPD inverse of k_bdf.hip and an FP64
// MFMA product (k_gemm.hip).
#include <algorithm>

#include "als.h"
#include "kcommon.h"

namespace rom {

// The right-hand sides go through two unfoldings of the tensor, rows of pitch np with zero
// padding:
//   layout 0: row (i, j), column k = C[i][j][k]   (C itself where N = np and it is aligned);
//   layout 1: row (j, k), column i = C[i][j][k].
// A product with one factor (FP64 MFMA) gives T[row][r], and an elementwise reduction with
// a second factor the right-hand side.
__global__ __launch_bounds__(256) void k_als_unfold(int N, int np, const double* __restrict__ C,
                                                    double* __restrict__ U, long long total) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= total) return;
    const long long row = q / np;
    const int c = (int)(q % np);
    U[q] = c < N ? C[row * N + c] : 0.0;
}

// Layout 1 is the transpose of the N x N^2 matrix C[i][(j, k)]: tiles of 32 i x 64 (j, k)
// through LDS, so both sides are read and written in runs of at least 256 bytes (read
// without the tiles, N = 200: 73 us; the copy of 2 x 64 MB itself 27).
__global__ __launch_bounds__(256) void k_als_unfold_t(int N, int np, const double* __restrict__ C,
                                                      double* __restrict__ U) {
    __shared__ double tile[32][65];
    const long long n2 = (long long)N * N, r0 = (long long)blockIdx.x * 64;
    const int i0 = blockIdx.y * 32, t = threadIdx.x;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int i = t / 64 + 4 * e;
        const long long jk = r0 + t % 64;
        tile[i][t % 64] = i0 + i < N && jk < n2 ? C[(size_t)(i0 + i) * n2 + jk] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int r = t / 32 + 8 * e, i = i0 + t % 32;
        if (r0 + r < n2 && i < np) U[(size_t)(r0 + r) * np + i] = tile[t % 32][r];
    }
}

void launch_als_unfold(int N, int np, int layout, const double* C, double* U, hipStream_t s) {
    if (layout == 1) {
        const unsigned gx = (unsigned)(((long long)N * N + 63) / 64);
        hipLaunchKernelGGL(k_als_unfold_t, dim3(gx, (unsigned)((np + 31) / 32)), dim3(256), 0, s, N, np, C, U);
        return;
    }
    const long long total = (long long)N * N * np;
    hipLaunchKernelGGL(k_als_unfold, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, N, np, C, U, total);
}

// Ft [R][np] = F^T with zero padding (the skinny product's operand rows).
__global__ __launch_bounds__(256) void k_als_transpose(int N, int R, int np, const double* __restrict__ F,
                                                       double* __restrict__ Ft) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long long)R * np) return;
    const int m = (int)(q / np), k = (int)(q % np);
    Ft[q] = k < N ? F[(size_t)k * R + m] : 0.0;
}

void launch_als_transpose(int N, int R, int np, const double* F, double* Ft, hipStream_t s) {
    const long long total = (long long)R * np;
    hipLaunchKernelGGL(k_als_transpose, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, N, R, np, F, Ft);
}

// T[b][m] = sum_k U[b][k] F[k][m] in FP64: the unfolding [Bn][np] times one factor [N][R],
// T [Bn][R].  A block keeps the factor's columns of G 16-column tiles in LDS for its whole
// life, in fragment order (one 16-byte vector per lane and 8-k step, zeros past N and R),
// and its eight wavefronts walk the 16-row tiles of the block's row range, w, w + 8, ...: a
// wavefront streams its U fragments straight from memory, four steps ahead and on into its
// next tile, and meets each with G tiles of the panel.  There is one block per compute unit
// (less those left to the inverse, see als_product_plan), ncg column groups x nrr row ranges
// (a row range's groups next to each other, so that one XCD's L2 serves them the same rows).
// Lane l feeds row l % 16 and, of an 8-k step, k = 2 (l / 16) + {0, 1} in both operands;
// accumulator element v of lane l is row l / 16 + 4 v and column l % 16.  Rows past Bn are
// clamped for the loads and not stored.
//
// Bound by the FP64 matrix rate.  With the rows in LDS and the factor streamed from L2 the
// product took 146 us on all compute units (N = 200, R = 400: 6.4 GFLOP), on 220 of 256 it
// takes 131; and the inverse's panels no longer wait for its blocks to retire (35 to 54 us
// each instead of 8).
template <int G>
__global__ __launch_bounds__(512) void k_als_product(int N, int R, int np, long long Bn, int ncg, int nrr,
                                                     const double* __restrict__ U, const double* __restrict__ F,
                                                     double* __restrict__ T) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    double2* fs = reinterpret_cast<double2*>(smem);      // [G][ks][64]
    const int per = (int)gridDim.x / 8, id = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    const int cg = id % ncg, rr = id / ncg;
    if (rr >= nrr) return;
    const int ks = np / 8, w = threadIdx.x / kWave, lane = threadIdx.x % kWave, g = lane >> 4, c16 = lane & 15;
    const int m0 = cg * G * 16;
    staged_copy<16, double2>(
        G * ks * kWave,
        [&](int q) {
            const int ln = q % kWave, st = (q / kWave) % ks, t = q / (kWave * ks);
            const int k = 8 * st + 2 * (ln / 16), m = m0 + 16 * t + ln % 16;
            double2 v = {0.0, 0.0};
            if (m < R && k < N) v.x = F[(size_t)k * R + m];
            if (m < R && k + 1 < N) v.y = F[(size_t)(k + 1) * R + m];
            return v;
        },
        [&](int q, const double2& v) { fs[q] = v; });
    __syncthreads();

    const long long tiles = (Bn + 15) / 16, tb = tiles * rr / nrr, te = tiles * (rr + 1) / nrr;
    constexpr int D = 4;                                 // steps in flight
    double2 ring[D];
    auto rowp = [&](long long u) {
        const long long b = u * 16 + c16;
        return U + (size_t)(b < Bn ? b : Bn - 1) * np + 2 * g;
    };
    long long u = tb + w;
    if (u >= te) return;
    const double* row = rowp(u);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (d < ks) ring[d] = *reinterpret_cast<const double2*>(row + 8 * d);
    }
    for (; u < te; u += 8) {
        f64x4 acc[G];
#pragma unroll
        for (int i = 0; i < G; ++i) acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};
        auto step = [&](int st, const double2& a) {
            double2 f[G];
#pragma unroll
            for (int i = 0; i < G; ++i) f[i] = fs[(i * ks + st) * kWave + lane];
#pragma unroll
            for (int i = 0; i < G; ++i) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, f[i].x, acc[i], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < G; ++i) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, f[i].y, acc[i], 0, 0, 0);
        };
        // whole rounds that refill every slot they consume (no branches), then the rest
        int s0 = 0;
        for (; s0 + 2 * D <= ks; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const double2 a = ring[d];
                ring[d] = *reinterpret_cast<const double2*>(row + 8 * (s0 + D + d));
                step(s0 + d, a);
            }
        }
#pragma unroll
        for (int d = 0; d < 2 * D - 1; ++d) {
            if (s0 + d >= ks) break;
            const double2 a = ring[d % D];
            if (s0 + D + d < ks) ring[d % D] = *reinterpret_cast<const double2*>(row + 8 * (s0 + D + d));
            step(s0 + d, a);
        }
        // the next tile's first steps, in flight behind this one's stores
        if (u + 8 < te) {
            row = rowp(u + 8);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (d < ks) ring[d] = *reinterpret_cast<const double2*>(row + 8 * d);
            }
        }
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int m = m0 + 16 * i + c16;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const long long b = u * 16 + g + 4 * v;
                if (b < Bn && m < R) T[b * R + m] = acc[i][v];
            }
        }
    }
}

namespace {

constexpr int kPanelTiles = 6;           // column tiles of a block, at most
// A panel may take a compute unit's whole LDS.  It reserves at least kPanelReserve, which
// leaves too little for a block of k_gj_step (27 KB): the inverse beside a product then runs
// on the compute units that the product's grid leaves it and never shares a unit with it.
// A product wavefront holds the SIMD's FP64 units 64 cycles an instruction, and a panel of
// the inverse beside it took 29 us instead of 8 (N = 200, R = 400: 6.9 ms for ten sweeps
// where they share the units, 5.8 where they don't; 8.4 with the product that staged rows).
constexpr size_t kPanelLds = 163840, kPanelReserve = 139264;

// the allowance of every plan: calls of different sizes may run at the same time
template <int G>
bool panel_ready() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_als_product<G>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPanelLds) == hipSuccess;
}

template <int G>
void panel_go(const AlsProductPlan& pl, int N, int R, int np, long long Bn, const double* U, const double* F, double* T,
              hipStream_t s) {
    const unsigned blocks = (unsigned)((pl.ncg * pl.nrr + 7) / 8 * 8);
    hipLaunchKernelGGL(k_als_product<G>, dim3(blocks), dim3(512), pl.lds, s, N, R, np, Bn, pl.ncg, pl.nrr, U, F, T);
}

}  // namespace

AlsProductPlan als_product_plan(int N, int R, int np) {
    AlsProductPlan pl{};
    const int nmt = (R + 15) / 16, ks = np / 8;
    const int gmax = (int)std::min<size_t>(kPanelTiles, kPanelLds / ((size_t)ks * kWave * sizeof(double2)));
    // one tile of columns is the least (the skinny GEMM that is left past it took three times as
    // long where both can run: N = R = 500, three sweeps 62 ms, here 21)
    if (gmax < 1) return pl;
    pl.ncg = (nmt + gmax - 1) / gmax;
    pl.g = (nmt + pl.ncg - 1) / pl.ncg;
    const long long tiles = ((long long)N * N + 15) / 16;
    // compute units per XCD left to the inverse: its nb^2 tiles in two rounds of three blocks a
    // unit (only one tile of a panel has more to do than two 32 x 32 products).  Ten sweeps at
    // N = 200, R = 400 (nb = 13): 7.4 ms with three units, 5.75 with 4 or 5, 5.9 with 6, 6.1
    // with 8.
    const int nb = (R + 31) / 32, cus = 32 - std::min(8, ((nb * nb + 7) / 8 + 5) / 6);
    pl.nrr = (int)std::max<long long>(1, std::min<long long>(tiles, 8 * cus / pl.ncg));
    pl.lds = std::max((size_t)pl.g * ks * kWave * sizeof(double2), kPanelReserve);
    switch (pl.g) {
        case 1: pl.ok = panel_ready<1>(); break;
        case 2: pl.ok = panel_ready<2>(); break;
        case 3: pl.ok = panel_ready<3>(); break;
        case 4: pl.ok = panel_ready<4>(); break;
        case 5: pl.ok = panel_ready<5>(); break;
        case 6: pl.ok = panel_ready<6>(); break;
    }
    if (!pl.ok) (void)hipGetLastError();    // a refused allowance is not the caller's error
    return pl;
}

void launch_als_product(const AlsProductPlan& pl, int N, int R, int np, long long Bn, const double* U, const double* F,
                        double* T, hipStream_t s) {
    switch (pl.g) {
        case 1: panel_go<1>(pl, N, R, np, Bn, U, F, T, s); break;
        case 2: panel_go<2>(pl, N, R, np, Bn, U, F, T, s); break;
        case 3: panel_go<3>(pl, N, R, np, Bn, U, F, T, s); break;
        case 4: panel_go<4>(pl, N, R, np, Bn, U, F, T, s); break;
        case 5: panel_go<5>(pl, N, R, np, Bn, U, F, T, s); break;
        case 6: panel_go<6>(pl, N, R, np, Bn, U, F, T, s); break;
    }
}

// M[p][r] (pitch ldm) = sum_q T[row(p, q)][r] F[q][r], row = p N + q (first index
// kept) or q N + p (second index kept); thread r, block row p.  T is streamed once (N^2 R
// values): eight rows are loaded before they are used, into eight partial sums added in a
// fixed order.
__global__ __launch_bounds__(256) void k_als_reduce(int N, int R, int keep_first, const double* __restrict__ T,
                                                    const double* __restrict__ F, double* __restrict__ M, int ldm) {
    const int p = blockIdx.y, r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    auto row = [&](int q) { return keep_first ? (size_t)p * N + q : (size_t)q * N + p; };
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int q = 0;
    for (; q + 8 <= N; q += 8) {
        double t[8], f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            t[e] = T[row(q + e) * R + r];
            f[e] = F[(size_t)(q + e) * R + r];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += t[e] * f[e];
    }
    for (; q < N; ++q) acc[0] += T[row(q) * R + r] * F[(size_t)q * R + r];
    M[(size_t)p * ldm + r] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
}

void launch_als_reduce(int N, int R, int keep_first, const double* T, const double* F, double* M, int ldm,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_als_reduce, dim3((R + 255) / 256, N), dim3(256), 0, s, N, R, keep_first, T, F, M, ldm);
}

// V = (Fa^T Fa) .* (Fb^T Fb) [R][R] on FP64 MFMA: a block per 32 x 32 tile of V, sixteen
// waves: wave w forms quarter w % 4 (rows r0, columns c0) over the factor rows of issues
// s = w / 4, w / 4 + 4, ... (four parts of the contracted range, added in LDS in a fixed
// order).  Lane l feeds row / column l % 16 and factor row k = 4 s + l / 16 of issue s, its
// operands read straight from the factors (16 consecutive values of one factor row per 16
// lanes); rows past N give zeros and columns past R are clamped for the loads and not
// stored.
constexpr int kGramParts = 4;
__global__ __launch_bounds__(256 * kGramParts) void k_gram_hadamard(int N, int R, const double* __restrict__ Fa,
                                                                   const double* __restrict__ Fb,
                                                                   double* __restrict__ V) {
    __shared__ f64x4 part[kGramParts - 1][4][kWave];
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave, qd = w % 4, kp = w / 4;
    const int r0 = blockIdx.y * 32 + (qd / 2) * 16, c0 = blockIdx.x * 32 + (qd % 2) * 16;
    const int rr = min(r0 + lane % 16, R - 1), cc = min(c0 + lane % 16, R - 1);
    f64x4 ga = {0.0, 0.0, 0.0, 0.0}, gb = {0.0, 0.0, 0.0, 0.0};
    const int steps = (N + 3) / 4;
#pragma unroll 4
    for (int st = kp; st < steps; st += kGramParts) {
        const int k = 4 * st + lane / 16;
        const bool in = k < N;
        const size_t o = (size_t)(in ? k : 0) * R;
        const double ar = in ? Fa[o + rr] : 0.0, ac = in ? Fa[o + cc] : 0.0;
        const double br = in ? Fb[o + rr] : 0.0, bc = in ? Fb[o + cc] : 0.0;
        ga = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, ac, ga, 0, 0, 0);
        gb = __builtin_amdgcn_mfma_f64_16x16x4f64(br, bc, gb, 0, 0, 0);
    }
    if (kp > 0) part[kp - 1][qd][lane] = ga;
    __syncthreads();
    if (kp == 0) {
#pragma unroll
        for (int q = 0; q < kGramParts - 1; ++q) ga += part[q][qd][lane];
    }
    __syncthreads();
    if (kp > 0) part[kp - 1][qd][lane] = gb;
    __syncthreads();
    if (kp > 0) return;
#pragma unroll
    for (int q = 0; q < kGramParts - 1; ++q) gb += part[q][qd][lane];
    // accumulator element v of lane l: row l / 16 + 4 v, column l % 16
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = r0 + lane / 16 + 4 * v, c = c0 + lane % 16;
        if (r < R && c < R) V[(size_t)r * R + c] = ga[v] * gb[v];
    }
}

void launch_gram_hadamard(int N, int R, const double* Fa, const double* Fb, double* V, hipStream_t s) {
    const unsigned t = (unsigned)((R + 31) / 32);
    hipLaunchKernelGGL(k_gram_hadamard, dim3(t, t), dim3(256 * kGramParts), 0, s, N, R, Fa, Fb, V);
}

// ---------------------------------------------------------------- ALS-skew (Sec. 3.3)
//
// Factors of the skew-symmetry preserving structure (eq. skew_abc_struct) with P column
// pairs, R = 2P: A1 = [A11 A12], A2 = [B1 B1], A3 = [A12 -A11], each [N][R].

// The three full factors from the blocks A11, A12, B1 [N][P].
__global__ void k_skew_assemble(int N, int P, const double* __restrict__ A11, const double* __restrict__ A12,
                                const double* __restrict__ B1, double* __restrict__ A1, double* __restrict__ A2,
                                double* __restrict__ A3) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long long)N * P) return;
    const int i = (int)(q / P), p = (int)(q % P);
    const size_t o = (size_t)i * 2 * P;
    const double a = A11[q], c = A12[q], b = B1[q];
    A1[o + p] = a;
    A1[o + P + p] = c;
    A2[o + p] = b;
    A2[o + P + p] = b;
    A3[o + p] = c;
    A3[o + P + p] = -a;
}

void launch_skew_assemble(int N, int P, const double* A11, const double* A12, const double* B1, double* A1,
                          double* A2, double* A3, hipStream_t s) {
    const long long n = (long long)N * P;
    hipLaunchKernelGGL(k_skew_assemble, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, N, P, A11, A12, B1, A1,
                       A2, A3);
}

// The normal equations of the tied second factor A2 = B1 S, S = [I; I]:
// Vt = S^T V S [P][P] from V [R][R], and Mt = M S [npad][ldt] from M [N][ldm]; a NULL V
// or M skips its part (the inverse of Vt can then start before M exists).
__global__ void k_skew_tie(int N, int P, const double* __restrict__ V, double* __restrict__ Vt,
                           const double* __restrict__ M, int ldm, double* __restrict__ Mt, int ldt) {
    const int row = blockIdx.y, p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const int R = 2 * P;
    if (row < P && V) {
        const double* v0 = V + (size_t)row * R;
        const double* v1 = V + (size_t)(P + row) * R;
        Vt[(size_t)row * P + p] = (v0[p] + v0[P + p]) + (v1[p] + v1[P + p]);
    }
    if (row < N && M) Mt[(size_t)row * ldt + p] = M[(size_t)row * ldm + p] + M[(size_t)row * ldm + P + p];
}

void launch_skew_tie(int N, int P, const double* V, double* Vt, const double* M, int ldm, double* Mt, int ldt,
                     hipStream_t s) {
    const int rows = N > P ? N : P;
    hipLaunchKernelGGL(k_skew_tie, dim3((P + 255) / 256, rows), dim3(256), 0, s, N, P, V, Vt, M, ldm, Mt, ldt);
}

// B1 from the tied solve Y [..][ldy] (first P columns), and A2 = [B1 B1].
__global__ void k_skew_set_b(int N, int P, const double* __restrict__ Y, int ldy, double* __restrict__ B1,
                             double* __restrict__ A2) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long long)N * P) return;
    const int i = (int)(q / P), p = (int)(q % P);
    const double b = Y[(size_t)i * ldy + p];
    B1[q] = b;
    A2[(size_t)i * 2 * P + p] = b;
    A2[(size_t)i * 2 * P + P + p] = b;
}

void launch_skew_set_b(int N, int P, const double* Y, int ldy, double* B1, double* A2, hipStream_t s) {
    const long long n = (long long)N * P;
    hipLaunchKernelGGL(k_skew_set_b, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, N, P, Y, ldy, B1, A2);
}

// Momentum update of the first factor from the subiteration's solution Y [..][ldy]:
// A1 <- mom A1 + (1 - mom) Y, the blocks A11, A12 written out, and A3 = [A12 -A11].
__global__ void k_skew_momentum(int N, int P, double mom, const double* __restrict__ Y, int ldy,
                                double* __restrict__ A1, double* __restrict__ A3, double* __restrict__ A11,
                                double* __restrict__ A12) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long long)N * P) return;
    const int i = (int)(q / P), p = (int)(q % P);
    const size_t o = (size_t)i * 2 * P;
    const double a = mom * A1[o + p] + (1.0 - mom) * Y[(size_t)i * ldy + p];
    const double c = mom * A1[o + P + p] + (1.0 - mom) * Y[(size_t)i * ldy + P + p];
    A1[o + p] = a;
    A1[o + P + p] = c;
    A3[o + p] = c;
    A3[o + P + p] = -a;
    A11[q] = a;
    A12[q] = c;
}

void launch_skew_momentum(int N, int P, double mom, const double* Y, int ldy, double* A1, double* A3, double* A11,
                          double* A12, hipStream_t s) {
    const long long n = (long long)N * P;
    hipLaunchKernelGGL(k_skew_momentum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, N, P, mom, Y, ldy, A1, A3,
                       A11, A12);
}

}  // namespace rom
