// k_contract.hip -- CP advection contraction for one trajectory.
//
// CP (Sec. 3.1, eq. tc_ap):  w = lam .* s .* t with s = Bf^T u, t = Cf^T u (one pass
// over [Bf | Cf]^T stored [2Rp][Np]: a wavefront takes rows r and Rp + r and writes w_r;
// factors with skew column pairs, Sec. 3.3, read the pair form instead), then y = Af w,
// with w staged in LDS by every block of the scatter kernel, which also applies the BDF
// update to its rows.  With a dense stiffness the Helmholtz kernel forms the next level's
// w.  The file also holds the first product of the SVD-ROM (Sec. 4.4).
// Np and Rp round N and R up to multiples of 8; padding rows and columns hold zeros
// (and zero weights), so they contribute nothing.
#include "kbody.h"

namespace rom {

// ============================================================== CP, one trajectory

template <int DT, int V, int U>
__global__ __launch_bounds__(256) void k_cp_proj1(Proj1Job jb) {
    cp_proj_any_body<DT, V, U>(jb, blockIdx.x);
}
// MODE 1 (the update kernel) runs one block more than there are row blocks: the last
// one closes the previous level and advances the counter.
template <int DT, int V, int U, int MODE, bool FULL>
__global__ __launch_bounds__(256) void k_cp_scatter1(Scat1Job jb, double* y_out) {
    if constexpr (MODE == 1) {
        if (blockIdx.x == gridDim.x - 1) {
            close_and_advance(jb.a, *jb.a.step, (int)gridDim.x - 1);
            return;
        }
        cp_scatter1_body<DT, V, U, MODE, FULL>(jb, y_out, blockIdx.x, *jb.a.step);
    } else {
        cp_scatter1_body<DT, V, U, MODE, FULL>(jb, y_out, blockIdx.x, MODE == 0 ? 0LL : *jb.a.step);
    }
}

// ============================================================== small evaluations
//
// y = Af (lam .* s .* t) of a small CP operator in one launch: every block forms all of w in
// LDS (each wavefront its share of the row pairs, four at a time) and then its own rows of
// y, so the second kernel, its launch and the trip of w through memory go; the price is the
// projection rows read by every block.  Dot products keep cp_proj1_body's, cp_proj_skew_body's
// and cp_scatter1_body's lane partition and order, so results are theirs to the bit.  Bound
// by latency: N = 37, R = 40 in FP64 took 3.7 us on the device against 5.3, and 4.8 us per
// call against 8.1.  A pair costs a wavefront about 0.5 us of reductions, so it is taken up to
// kSmallMost pairs (R = 80 in pair form) and kSmallBytes of projection rows: N = R = 64 in
// FP64 4.8 against 5.3 us, N = 50, R = 100 6.5 against 5.3.  Blocks write y while others read u,
// so the two arrays must not share memory (the two launches serve those that do).
constexpr size_t kSmallBytes = 48 << 10;
constexpr int kSmallWaves = 16, kSmallMost = 40;
template <int DT> constexpr int kSmallPairs = DT == DT_BF16X3 ? 2 : 4;

template <int DT, int V, int NR>
__device__ __forceinline__ void cp_w_in_lds(const Proj1Job& jb, const LdsU<DT>& L, const LdsU<DT>& Ln,
                                            typename Store<DT>::Acc* W) {
    typedef typename Store<DT>::T T;
    typedef typename Store<DT>::Acc Acc;
    constexpr bool X3 = (DT == DT_BF16X3), NEGU = (DT == DT_BF16 || DT == DT_BF16X3);
    typedef typename RawT<V * (int)sizeof(T)>::T Raw;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int Np = jb.Np, P = jb.P, np = NR == 3 ? P : jb.Rp, k = lane * V;
    const T* op = reinterpret_cast<const T*>(jb.BCt);
    const Acc* lam = reinterpret_cast<const Acc*>(jb.lam);
    auto cols = [&](int q, int& c0, int& c1) {
        c0 = jb.layout == 1 ? 2 * q : q;
        c1 = jb.layout == 1 ? 2 * q + 1 : P + q;
    };
    Raw rv[kSmallPairs<DT>][NR], rl[kSmallPairs<DT>][NR];
    Acc lv[kSmallPairs<DT>][2];
    auto issue = [&](int q0) {
#pragma unroll
        for (int e = 0; e < kSmallPairs<DT>; ++e) {
            const int q = q0 + e * kSmallWaves;
            if (q >= np) continue;
            int c0, c1;
            cols(q, c0, c1);
            const int rows[3] = {q, NR == 3 ? P + c0 : jb.Rp + q, P + c1};
            lv[e][0] = lam[NR == 3 ? c0 : q];
            lv[e][1] = NR == 3 ? lam[c1] : 0;
#pragma unroll
            for (int h = 0; h < NR; ++h)
                if (k < Np) {
                    rv[e][h] = ld_plain<V * (int)sizeof(T)>(op + (size_t)rows[h] * Np + k);
                    if constexpr (X3) rl[e][h] = ld_plain<V * (int)sizeof(T)>(jb.BCt_lo + (size_t)rows[h] * Np + k);
                }
        }
    };
    issue(w);
    L.fill(jb.u_base, jb.N, Np);
    if constexpr (NEGU && NR == 3) Ln.fill(jb.u_base, jb.N, Np, -1.0);
    __syncthreads();
    for (int q0 = w; q0 < np; q0 += kSmallPairs<DT> * kSmallWaves) {
        if (q0 != w) issue(q0);
#pragma unroll
        for (int e = 0; e < kSmallPairs<DT>; ++e) {
            const int q = q0 + e * kSmallWaves;
            if (q >= np) continue;
            Acc z[NR];
#pragma unroll
            for (int h = 0; h < NR; ++h) {
                z[h] = 0;
                if (k < Np) z[h] += dot_vec<DT, V>(rv[e][h], rl[e][h], NEGU && NR == 3 && h == 1 ? Ln : L, k);
                z[h] = wave_sum(z[h]);
            }
            if (lane == 0) {
                if constexpr (NR == 3) {
                    int c0, c1;
                    cols(q, c0, c1);
                    W[c0] = lv[e][0] * z[0] * z[2];
                    W[c1] = lv[e][1] * z[0] * (NEGU ? z[1] : -z[1]);
                } else {
                    W[q] = lv[e][0] * z[0] * z[1];
                }
            }
        }
    }
    if (NR == 3 && (int)threadIdx.x < jb.Rp - jb.R) W[jb.R + threadIdx.x] = 0;   // padding past R
}

template <int DT, int V>
__global__ __launch_bounds__(64 * kSmallWaves) void k_cp_eval_small(Proj1Job pj, Scat1Job sj, double* __restrict__ y) {
    typedef typename Store<DT>::T T;
    typedef typename Store<DT>::Acc Acc;
    constexpr bool X3 = (DT == DT_BF16X3), NEGU = (DT == DT_BF16 || DT == DT_BF16X3);
    typedef typename RawT<V * (int)sizeof(T)>::T Raw;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const size_t ub = LdsU<DT>::bytes(pj.Np);
    LdsU<DT> L, Ln;
    L.bind(smem, pj.Np);
    Ln.bind(smem + (NEGU ? ub : 0), pj.Np);
    Acc* W = reinterpret_cast<Acc*>(smem + (NEGU ? 2 : 1) * ub);
    const int lane = threadIdx.x % kWave, i = (int)blockIdx.x * kSmallWaves + threadIdx.x / kWave;
    const int R = sj.Rp;
    const bool live = i < sj.N;
    // the wavefront's row of Af, ahead of the projections
    Raw rv, rl;
    const int r = lane * V;
    if (live && r < R) {
        rv = ld_plain<V * (int)sizeof(T)>(reinterpret_cast<const T*>(sj.Af) + (size_t)i * R + r);
        if constexpr (X3) rl = ld_plain<V * (int)sizeof(T)>(sj.Af_lo + (size_t)i * R + r);
    }
    if (pj.layout) cp_w_in_lds<DT, V, 3>(pj, L, Ln, W);
    else cp_w_in_lds<DT, V, 2>(pj, L, Ln, W);
    __syncthreads();
    if (!live) return;
    Acc z = 0;
    if (r < R) {
        Acc cv[V];
        Decode<DT, V>::run(rv, cv);
        if constexpr (X3) {
            float cl[V];
            Decode<DT, V>::run(rl, cl);
#pragma unroll
            for (int v = 0; v < V; ++v) z += (cv[v] + cl[v]) * W[r + v];
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) z += cv[v] * W[r + v];
        }
    }
    z = wave_sum(z);
    if (lane == 0) y[i] = (double)z;
}

// ============================================================== Helmholtz apply and projections

// One state: nh + np blocks and a last one that closes the previous level and advances
// the counter.
template <int DT, bool EVEN>
__global__ __launch_bounds__(256) void k_helm_proj(HelmJob jb) {
    if (blockIdx.x == gridDim.x - 1) {
        close_and_advance(jb.a, *jb.a.step, jb.nh);
        return;
    }
    helm_proj_body<DT, EVEN>(jb, *jb.a.step, blockIdx.x);
}

// ============================================================== SVD-ROM, one trajectory

// First product of the SVD-ROM, one state (svd_proj_body).
template <int DT, int V, int U>
__global__ __launch_bounds__(256) void k_svd_proj(SvdProj a) {
    svd_proj_body<DT, V, U>(a, (int)blockIdx.x);
}

template <int DT>
static void svd_proj_go(const SvdProj& a, hipStream_t s) {
    constexpr int V = 16 / (int)sizeof(typename Store<DT>::T);
    hipLaunchKernelGGL((k_svd_proj<DT, V, 4>), dim3((unsigned)((a.Rsp + 3) / 4)), dim3(256), LdsU<DT>::bytes(a.Np), s,
                       a);
}

void launch_svd_proj(int dt, const void* Ut, const void* Ut_lo, const void* sigma, int N, int Np, int Rs,
                     const double* u_base, const long long* stepp, long long slot_stride, void* w, hipStream_t s) {
    SvdProj a{};
    a.Ut = Ut;
    a.Ut_lo = (const unsigned short*)Ut_lo;
    a.sigma = sigma;
    a.N = N;
    a.Np = Np;
    a.Rsp = (Rs + 7) / 8 * 8;
    a.u_base = u_base;
    a.stepp = stepp;
    a.slot_stride = slot_stride;
    a.w = w;
    switch (dt) {
        case DT_F64: svd_proj_go<DT_F64>(a, s); break;
        case DT_F32: svd_proj_go<DT_F32>(a, s); break;
        case DT_BF16: svd_proj_go<DT_BF16>(a, s); break;
        default: svd_proj_go<DT_BF16X3>(a, s); break;
    }
}

// ---------------------------------------------------------------- launchers

// LDS of the projection kernels: the image of u, and for the BF16 formats a second one
// of -u (read by the pair form).
template <int DT>
static size_t proj_lds(int Np) {
    return (DT == DT_BF16 || DT == DT_BF16X3 ? 2 : 1) * LdsU<DT>::bytes(Np);
}

template <int DT>
static void proj1_go(const Proj1Job& jb, hipStream_t s) {
    constexpr int V = 16 / (int)sizeof(typename Store<DT>::T);
    hipLaunchKernelGGL((k_cp_proj1<DT, V, 4>), dim3((unsigned)jb.nblk), dim3(256), proj_lds<DT>(jb.Np), s, jb);
}

static void proj1_dispatch(int dt, const Proj1Job& jb, hipStream_t s) {
    switch (dt) {
        case DT_F64: proj1_go<DT_F64>(jb, s); break;
        case DT_F32: proj1_go<DT_F32>(jb, s); break;
        case DT_BF16: proj1_go<DT_BF16>(jb, s); break;
        default: proj1_go<DT_BF16X3>(jb, s); break;
    }
}

// Blocks of the projection kernel: four row pairs of [Bf|Cf]^T, or four column pairs
// of the pair form, per block.
int proj1_blocks(int Rp, SkewPairs sk) { return sk.layout ? (Rp / 2 + 3) / 4 : (Rp + 3) / 4; }

static Proj1Job proj1_job(const void* BCt, const void* BCt_lo, const void* lam, int N, int Np, int Rp, SkewPairs sk,
                          const double* u_base, const long long* stepp, long long slot_stride, void* w) {
    Proj1Job jb{};
    jb.BCt = BCt;
    jb.BCt_lo = (const unsigned short*)BCt_lo;
    jb.lam = lam;
    jb.N = N;
    jb.Np = Np;
    jb.Rp = Rp;
    jb.layout = sk.layout;
    jb.P = sk.P;
    jb.R = sk.R;
    jb.u_base = u_base;
    jb.stepp = stepp;
    jb.slot_stride = slot_stride;
    jb.w = w;
    jb.nblk = proj1_blocks(Rp, sk);
    return jb;
}

int launch_cp_proj1(int dt, const void* BCt, const void* BCt_lo, const void* lam, int N, int Np, int Rp,
                    SkewPairs sk, const double* u_base, const long long* stepp, long long slot_stride,
                    void* w, hipStream_t s) {
    proj1_dispatch(dt, proj1_job(BCt, BCt_lo, lam, N, Np, Rp, sk, u_base, stepp, slot_stride, w), s);
    return 0;
}

template <int DT>
static void eval_small_go(const Proj1Job& pj, const Scat1Job& sj, double* y, hipStream_t s) {
    constexpr int V = 16 / (int)sizeof(typename Store<DT>::T);
    const size_t lds = proj_lds<DT>(pj.Np) + sizeof(typename Store<DT>::Acc) * (size_t)pj.Rp;
    hipLaunchKernelGGL((k_cp_eval_small<DT, V>), dim3((unsigned)((sj.N + kSmallWaves - 1) / kSmallWaves)),
                       dim3(64 * kSmallWaves), lds, s, pj, sj, y);
}

bool launch_cp_eval_small(int dt, const void* BCt, const void* BCt_lo, const void* lam, const void* Af, const void* Af_lo,
                          int N, int Np, int Rp, SkewPairs sk, const double* u, double* y, hipStream_t s) {
    const int eb = dt == DT_F64 ? 8 : dt == DT_F32 ? 4 : 2, V = 16 / eb;
    const size_t rows = sk.layout ? (size_t)sk.P + sk.R : (size_t)2 * Rp;
    const size_t bytes = rows * Np * (dt == DT_BF16X3 ? 4 : eb);
    // one lane vector per row
    if (Np > kWave * V || Rp > kWave * V || (sk.layout ? sk.P : Rp) > kSmallMost || bytes > kSmallBytes) return false;
    const Proj1Job pj = proj1_job(BCt, BCt_lo, lam, N, Np, Rp, sk, u, nullptr, 0, nullptr);
    Scat1Job sj{};
    sj.Af = Af;
    sj.Af_lo = (const unsigned short*)Af_lo;
    sj.N = N;
    sj.Rp = Rp;
    switch (dt) {
        case DT_F64: eval_small_go<DT_F64>(pj, sj, y, s); break;
        case DT_F32: eval_small_go<DT_F32>(pj, sj, y, s); break;
        case DT_BF16: eval_small_go<DT_BF16>(pj, sj, y, s); break;
        default: eval_small_go<DT_BF16X3>(pj, sj, y, s); break;
    }
    return true;
}

template <int DT, int MODE>
static void scat1_go(const Scat1Job& jb, double* y, hipStream_t s) {
    typedef typename Store<DT>::Acc Acc;
    constexpr int V = 16 / (int)sizeof(typename Store<DT>::T);
    const dim3 grid((unsigned)jb.nblk + (MODE == 1 ? 1u : 0u));
    const size_t w_lds = sizeof(Acc) * jb.Rp;
    if (MODE != 0 && jb.G) {
        // W, then [uhat; h] (2 Np doubles) 16-byte aligned behind it
        const size_t lds = ((w_lds + 15) & ~(size_t)15) + sizeof(double) * 2 * jb.a.Np;
        hipLaunchKernelGGL((k_cp_scatter1<DT, V, 8, MODE, MODE != 0>), grid, dim3(256), lds, s, jb, y);
    } else {
        hipLaunchKernelGGL((k_cp_scatter1<DT, V, 8, MODE, false>), grid, dim3(256), w_lds, s, jb, y);
    }
}

template <int DT>
static void scat1_mode(int mode, const Scat1Job& jb, double* y, hipStream_t s) {
    if (mode == 0) scat1_go<DT, 0>(jb, y, s);
    else if (mode == 1) scat1_go<DT, 1>(jb, y, s);
    else scat1_go<DT, 2>(jb, y, s);
}

static void scat1_dispatch(int dt, int mode, const Scat1Job& jb, double* y, hipStream_t s) {
    switch (dt) {
        case DT_F64: scat1_mode<DT_F64>(mode, jb, y, s); break;
        case DT_F32: scat1_mode<DT_F32>(mode, jb, y, s); break;
        case DT_BF16: scat1_mode<DT_BF16>(mode, jb, y, s); break;
        default: scat1_mode<DT_BF16X3>(mode, jb, y, s); break;
    }
}

int launch_cp_scatter1(int dt, const void* Af, const void* Af_lo, int N, int Rp, const void* w, double* y_out,
                       const StepArgs* sa, int mode, hipStream_t s, const double* G) {
    Scat1Job jb{};
    jb.G = G;
    jb.Af = Af;
    jb.Af_lo = (const unsigned short*)Af_lo;
    jb.N = N;
    jb.Rp = Rp;
    jb.w = w;
    if (sa) jb.a = *sa;
    jb.nblk = (N + 3) / 4;
    scat1_dispatch(dt, mode, jb, y_out, s);
    return 0;
}

template <int DT>
static size_t helm_proj_lds(int N, int Np, bool proj) {
    // projections: images of u and (BF16 formats, pair form) -u
    const size_t h = sizeof(double) * (size_t)N, q = proj ? proj_lds<DT>(Np) : 0;
    return h > q ? h : q;
}

template <int DT>
static void helm_proj_go(const HelmJob& jb, hipStream_t s) {
    const size_t lds = helm_proj_lds<DT>(jb.a.N, jb.a.Np, jb.np > 0);
    const unsigned blocks = (unsigned)(jb.nh + jb.np + 1);
    if (jb.a.N % 2 == 0) hipLaunchKernelGGL((k_helm_proj<DT, true>), dim3(blocks), dim3(256), lds, s, jb);
    else hipLaunchKernelGGL((k_helm_proj<DT, false>), dim3(blocks), dim3(256), lds, s, jb);
}

void launch_helm_proj(int dt, const HelmJob& jb, hipStream_t s) {
    switch (dt) {
        case DT_F64: helm_proj_go<DT_F64>(jb, s); break;
        case DT_F32: helm_proj_go<DT_F32>(jb, s); break;
        case DT_BF16: helm_proj_go<DT_BF16>(jb, s); break;
        default: helm_proj_go<DT_BF16X3>(jb, s); break;
    }
}

}  // namespace rom
