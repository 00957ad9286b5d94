// k_fold.hip -- the dense advection contraction over the folded tensor (kfold.h): staging,
// the one-trajectory stream and the batched product on the matrix cores.
//
// Batched (k_fold_mm):  Y[b][i] = sum_c sum_{j in J(c)} S[j][b] sum_{k in c} F[i][j][k] X[b][k]
// with X = u in the MFMA operand format and S = u in the accumulation format.  The MFMA
// operand built from X over chunk c does not depend on j: a wavefront loads its X
// fragments once per chunk, keeps them in registers and streams the chunk's slabs through a
// prefetch ring, weighting each finished 16 x 16 tile by the j-weights of its trajectories
// (VALU).  Block = 4 wavefronts over 16 rows and 16*FN trajectories; the wavefronts take
// every fourth slab of a piece (chunk, part of its j range), so a block streams one
// contiguous run and the work splits evenly whatever N is (k_kr cuts k over the wavefronts:
// 4/3/3/3 steps at N = 400).  A block walks `ppb` consecutive pieces,
// accumulating in registers, then adds its wavefronts' tiles in LDS in a fixed order and
// writes one partial tile part[split][b][i], which the consumer sums in order.
//
// Bounds and times against the unfolded kernels these replaced: large batches by the matrix
// cores (N = 400, B = 256: FP32 155 us, 114 TFLOP/s of the 17.7 GFLOP left, 289 unfolded;
// BF16X3 55-61 against 97; FP64 at B = 64 82, 54 TFLOP/s), small ones and one trajectory by
// HBM (BF16X3 at N = 700, B = 16: 111 us, 6.8 TB/s, 230 unfolded; FP32 at N = 1000, one
// trajectory: 301 us, 6.9 TB/s, 574 unfolded), small tensors by latency (N = 100, one
// trajectory: 3.7 us against 11.5).
#include <type_traits>

#include "kfold.h"
#include "kmfma.h"

namespace rom {

typedef __attribute__((address_space(1))) void* gptr_t;   // global (HBM) pointer
typedef __attribute__((address_space(3))) void* lptr_t;   // LDS pointer

// ---------------------------------------------------------------- staging

// Rows i0 .. i0 + ni - 1 of the FP64 tensor (src = C[i0][0][0], row-major) into the folded
// storage.  Block (q-block of 32 slabs, chunk, row): both orientations of the 32 x kc patch
// of C[i] are read along their rows, the transposed one through LDS.  *flag is raised when a
// word of a folded tensor is not finite (the caller then stages it unfolded).  SVD: src holds
// V[i][k][r], whose slabs are the r.
template <int DT, bool SVD>
__global__ __launch_bounds__(256) void k_fold_pack(const double* __restrict__ src, int i0, FoldLay l, void* dst,
                                                   unsigned short* dst_lo, int* flag) {
    typedef typename Store<DT>::T T;
    constexpr int VEC = FoldT<DT>::VEC, KC = FoldT<DT>::KS * FoldT<DT>::KW, QB = 32;
    __shared__ double tr[KC][QB + 1];
    const int c = blockIdx.y, i = i0 + (int)blockIdx.z, qb = blockIdx.x * QB;
    int js, len;
    fold_range(l, c, js, len);
    if (qb >= len) return;
    const double* __restrict__ Ci = src + (size_t)blockIdx.z * l.N * l.J;
    const int k0 = c * KC, N = l.N;
    auto jof = [&](int q) {
        const int j = js + q;
        return j < N ? j : j - N;
    };
    if (SVD || l.fold) {
        for (int e = threadIdx.x; e < KC * QB; e += 256) {
            const int kk = e / QB, q = e - kk * QB;
            tr[kk][q] = (qb + q < len && k0 + kk < N) ? Ci[(size_t)(k0 + kk) * l.J + (SVD ? qb + q : jof(qb + q))] : 0.0;
        }
        __syncthreads();
    }
    const int width = fold_width(l, c);
    const size_t base = fold_base(l, i / 16, c);
    bool bad = false;
    for (int e = threadIdx.x; e < QB * (KC / VEC); e += 256) {
        const int q = e / (KC / VEC), ku = e - q * (KC / VEC);
        if (qb + q >= len || ku * VEC >= width) continue;
        const int j = SVD ? 0 : jof(qb + q);
        T hi[VEC];
        unsigned short lo[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const int kk = ku * VEC + v, k = k0 + kk;
            double x = 0.0;
            if (SVD) {
                x = tr[kk][q];
            } else if (k < N) {
                const double a = Ci[(size_t)j * N + k];
                if (!l.fold || k == j) x = a;
                else if (j < k0 || j >= k0 + KC || k > j) x = a + tr[kk][q];
            }
            if constexpr (DT == DT_F64) {
                hi[v] = x;
                bad |= !isfinite(x);
            } else if constexpr (DT == DT_F32) {
                hi[v] = (float)x;
                bad |= !isfinite((float)x);
            } else {
                const float f = (float)x;
                hi[v] = bf16_bits(f);
                if constexpr (DT == DT_BF16X3) lo[v] = bf16_bits(f - bf16_f(hi[v]));
                bad |= !isfinite(bf16_f(hi[v]));
            }
        }
        const size_t o = base + (size_t)(qb + q) * width * 16 + ((size_t)ku * 16 + (i & 15)) * VEC;
        *reinterpret_cast<u32x4*>(reinterpret_cast<T*>(dst) + o) = *reinterpret_cast<const u32x4*>(hi);
        if constexpr (DT == DT_BF16X3)
            *reinterpret_cast<u32x4*>(dst_lo + o) = *reinterpret_cast<const u32x4*>(lo);
    }
    if (l.fold && bad) *flag = 1;
}

static int fold_kc(int dt) { return dt == DT_BF16 || dt == DT_BF16X3 ? 64 : 32; }

FoldLay fold_layout(int dt, int N, int J, bool fold) {
    FoldLay l{};
    l.N = N;
    l.J = J;
    l.kc = fold_kc(dt);
    l.nk = (N + l.kc - 1) / l.kc;
    l.fold = fold ? 1 : 0;
    l.lmax = 0;
    for (int c = 0; c < l.nk; ++c) {
        int js, len;
        fold_range(l, c, js, len);
        l.lmax = len > l.lmax ? len : l.lmax;
    }
    return l;
}

size_t fold_elems(const FoldLay& l) { return (size_t)((l.N + 15) / 16) * l.nk * l.lmax * l.kc * 16; }

template <int DT>
static void fold_pack_go(bool svd, dim3 grid, hipStream_t s, const double* src, int i0, const FoldLay& l, void* dst,
                         unsigned short* lo, int* flag) {
    if (svd) hipLaunchKernelGGL((k_fold_pack<DT, true>), grid, dim3(256), 0, s, src, i0, l, dst, lo, flag);
    else hipLaunchKernelGGL((k_fold_pack<DT, false>), grid, dim3(256), 0, s, src, i0, l, dst, lo, flag);
}

void launch_fold_pack(int dt, bool svd, const double* src, int i0, int ni, const FoldLay& l, void* dst, void* dst_lo,
                      int* flag, hipStream_t s) {
    const dim3 grid((unsigned)((l.lmax + 31) / 32), (unsigned)l.nk, (unsigned)ni);
    unsigned short* lo = (unsigned short*)dst_lo;
    switch (dt) {
        case DT_F64: fold_pack_go<DT_F64>(svd, grid, s, src, i0, l, dst, lo, flag); break;
        case DT_F32: fold_pack_go<DT_F32>(svd, grid, s, src, i0, l, dst, lo, flag); break;
        case DT_BF16: fold_pack_go<DT_BF16>(svd, grid, s, src, i0, l, dst, lo, flag); break;
        default: fold_pack_go<DT_BF16X3>(svd, grid, s, src, i0, l, dst, lo, flag); break;
    }
}

// ---------------------------------------------------------------- one trajectory

template <int DT, bool NT>
__global__ __launch_bounds__(256) void k_fold_gemv(FoldJob jb) {
    fold_gemv_body<DT, kFoldU, NT>(jb, blockIdx.x);
}

// Bytes of the folded words, and whether they outgrow the 256 MB last-level cache: such a
// tensor streams past it with non-temporal loads (one trajectory, FP32 at N = 700: 110 us
// against 125), a smaller one is read from it step after step (N = 400: 22 us against 25).
static double fold_bytes(int dt, const FoldLay& l) {
    return (double)l.N * l.nk * l.lmax * l.kc * (dt == DT_F64 ? 8 : dt == DT_BF16 ? 2 : 4);
}
static bool fold_streams(int dt, const FoldLay& l) { return fold_bytes(dt, l) > 200e6; }

// Pieces per chunk: about `target` blocks in all, at least 4 slabs per wavefront.
int fold_gemv_njr(const FoldLay& l, int target) {
    const long long base = (long long)((l.N + 15) / 16) * l.nk;
    long long njr = (target + base - 1) / base;
    const long long most = (l.lmax + 15) / 16;
    if (njr > most) njr = most;
    return njr < 1 ? 1 : (int)njr;
}

FoldJob make_fold_job(int dt, const void* C, const void* Clo, const FoldLay& l, const void* wj, const double* u_base, const long long* stepp,
                      long long slot_stride, void* part, int njr) {
    FoldJob jb{};
    jb.C = C;
    jb.Clo = (const unsigned short*)Clo;
    jb.l = l;
    jb.wj = wj;
    jb.u_base = u_base;
    jb.stepp = stepp;
    jb.slot_stride = slot_stride;
    jb.part = part;
    jb.njr = njr;
    jb.jc = (l.lmax + njr - 1) / njr;
    jb.stream = fold_streams(dt, l) ? 1 : 0;
    jb.nblk = (l.N + 15) / 16 * l.nk * njr;
    return jb;
}

size_t fold_gemv_lds(int dt, const FoldJob& jb) { return (size_t)(jb.jc + 1) * (dt == DT_F64 ? 8 : 4); }

template <int DT>
static void fold_gemv_go(const FoldJob& jb, size_t lds, hipStream_t s) {
    const dim3 grid((unsigned)jb.nblk);
    if (jb.stream) hipLaunchKernelGGL((k_fold_gemv<DT, true>), grid, dim3(256), lds, s, jb);
    else hipLaunchKernelGGL((k_fold_gemv<DT, false>), grid, dim3(256), lds, s, jb);
}

void launch_fold_gemv(int dt, const FoldJob& jb, hipStream_t s) {
    const size_t lds = fold_gemv_lds(dt, jb);
    switch (dt) {
        case DT_F64: fold_gemv_go<DT_F64>(jb, lds, s); break;
        case DT_F32: fold_gemv_go<DT_F32>(jb, lds, s); break;
        case DT_BF16: fold_gemv_go<DT_BF16>(jb, lds, s); break;
        default: fold_gemv_go<DT_BF16X3>(jb, lds, s); break;
    }
}

// ---------------------------------------------------------------- batches

struct FoldArgs {
    const void* C;                 // folded tensor, storage format
    const unsigned short* Clo;     // BF16X3 low words
    const void* X;                 // [Bpad][Kx] coefficients in the MFMA operand format
    const unsigned short* Xlo;     // BF16X3 low words of X
    const void* S;                 // [N][Bpad] j-weights (FP64 for FP64, else FP32)
    void* part;                    // [nsplit][Bpad][N] partial tiles (accumulation type)
    FoldLay l;
    int Kx, Bpad;
    int njr, jc, ppb;              // pieces per chunk, slabs per piece, pieces per block
    int sp0, nsplit;               // first partial tile, their number: blocks per tile
    int gx, gy;
};

template <int FN, class Acc>
__device__ __forceinline__ void lds_row(const Acc* p, Acc (&v)[FN]) {
    constexpr int EV = 16 / (int)sizeof(Acc);
    if constexpr (FN % EV == 0) {
#pragma unroll
        for (int q = 0; q < FN / EV; ++q) {
            const u32x4 x = reinterpret_cast<const u32x4*>(p)[q];
            const Acc* e = reinterpret_cast<const Acc*>(&x);
#pragma unroll
            for (int i = 0; i < EV; ++i) v[q * EV + i] = e[i];
        }
    } else {
#pragma unroll
        for (int t = 0; t < FN; ++t) v[t] = p[t];
    }
}

template <int DT> struct FoldMk;
template <> struct FoldMk<DT_F64> { static constexpr int mk = MK_F64; };
template <> struct FoldMk<DT_F32> { static constexpr int mk = MK_F32; };
template <> struct FoldMk<DT_BF16X3> { static constexpr int mk = MK_BF16X3; };

template <int DT, int FN, int PF, bool NT>
__global__ __launch_bounds__(256) void k_fold_mm(FoldArgs p) {
    constexpr int MKD = FoldMk<DT>::mk;
    typedef MfmaT<MKD> Tr;
    typedef typename Tr::X XT;
    typedef typename Tr::Acc Acc;
    typedef typename Tr::Acc4 Acc4;
    typedef typename Store<DT>::T AT;
    constexpr int KS = FoldT<DT>::KS, VEC = FoldT<DT>::VEC, KW = FoldT<DT>::KW, NC = 16 * FN;
    constexpr int EV = 16 / (int)sizeof(Acc);
    constexpr bool X3 = (DT == DT_BF16X3);
    static_assert(KS == Tr::KS && VEC == Tr::VEC, "slab steps are MFMA steps");
    static_assert(1024 % (NC * (int)sizeof(Acc)) == 0, "a j-weight row must divide a 1 KB chunk");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    Acc* sl = reinterpret_cast<Acc*>(smem);              // [nq + 1][NC] j-weights, row nq zero

    // XCD-aware decode: consecutive block ids go round-robin over the 8 XCDs, so ids
    // q, q+8, ... (one XCD) take consecutive work items; the column tiles of one (row tile,
    // split) are consecutive and share that XCD's L2 for their tensor reads.
    const int nwork = p.gx * p.gy * p.nsplit;
    const int per = (nwork + 7) / 8;
    const int wi = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (wi >= nwork) return;
    const int by = wi % p.gy, sp = (wi / p.gy) % p.nsplit, bx = wi / (p.gy * p.nsplit);

    const FoldLay& l = p.l;
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b0 = by * NC;
    const int piece0 = (p.sp0 + sp) * p.ppb;
    const int piece1 = piece0 + p.ppb < l.nk * p.njr ? piece0 + p.ppb : l.nk * p.njr;

    Acc4 Y[FN];
#pragma unroll
    for (int t = 0; t < FN; ++t) Y[t] = Acc4{0, 0, 0, 0};

    for (int piece = piece0; piece < piece1; ++piece) {
        const int c = piece / p.njr, jr = piece - c * p.njr;
        int js, len;
        fold_range(l, c, js, len);
        const int q0 = jr * p.jc, q1 = q0 + p.jc < len ? q0 + p.jc : len;
        const int nq = q1 - q0;
        if (nq <= 0) continue;                           // block-uniform
        const int width = fold_width(l, c);

        __syncthreads();                                 // the previous piece's weights are no longer read
        // ---- the piece's j-weights straight into LDS: wavefront w copies the 1 KB chunks
        // w, w+4, ... of the [nq][NC] rows.  Columns past Bpad read a valid weight (their X
        // fragments are zero and their columns are never stored).
        {
            constexpr int rowb = NC * (int)sizeof(Acc);
            constexpr int rpc = 1024 / rowb;
            const int nch = (nq + rpc - 1) / rpc;
            const int r_in = (lane * 16) / rowb, cb = (lane * 16) % rowb;
            const int col = cb / (int)sizeof(Acc);
            const int colc = b0 + col < p.Bpad ? col : 0;
            for (int ch = w; ch < nch; ch += 4) {
                const int qq = ch * rpc + r_in;
                if (qq < nq) {
                    int j = js + q0 + qq;
                    j = j < l.N ? j : j - l.N;
                    const Acc* src = reinterpret_cast<const Acc*>(p.S) + (size_t)j * p.Bpad + b0 + colc;
                    __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(smem + (size_t)ch * 1024), 16, 0, 0);
                }
            }
            for (int e = threadIdx.x; e < NC / EV; e += 256)
                *reinterpret_cast<u32x4*>(sl + (size_t)nq * NC + e * EV) = u32x4{0u, 0u, 0u, 0u};
        }

        auto run = [&](auto nsc) {
            constexpr int NS = decltype(nsc)::value;
            // X fragments of the chunk for the lane's trajectories (column c16 of tile t is
            // trajectory b0 + c16*FN + t), zero past Kx or Bpad (addresses clamped)
            u32x4 xh[NS][FN], xl[NS][FN];
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int t = 0; t < FN; ++t) {
                    const int k = c * l.kc + s * KS + g * VEC;
                    const int b = b0 + c16 * FN + t;
                    const size_t o = (size_t)(b < p.Bpad ? b : p.Bpad - 1) * p.Kx + (k < p.Kx ? k : p.Kx - VEC);
                    xh[s][t] = ld_plain<16>(reinterpret_cast<const XT*>(p.X) + o);
                    if constexpr (X3) xl[s][t] = ld_plain<16>(p.Xlo + o);
                    else xl[s][t] = u32x4{0u, 0u, 0u, 0u};
                }
            lds_loads_done();                            // the weights
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int t = 0; t < FN; ++t) {
                    const int k = c * l.kc + s * KS + g * VEC;
                    const int b = b0 + c16 * FN + t;
                    if (!(k < p.Kx && b < p.Bpad)) {
                        xh[s][t] = u32x4{0u, 0u, 0u, 0u};
                        xl[s][t] = u32x4{0u, 0u, 0u, 0u};
                    }
                }

            // prefetch ring of PF slabs in rounds without branches whose loads are not predicated
            // (slabs past the end repeat the last one and meet the zero weight row), so the
            // compiler waits for the slot it consumes only.  With one column tile per block
            // (small problems, few slabs) the last slabs are consumed without loads behind them
            // (N = 64, B = 7: 3.4 us against 4.1); the wider tiles are bound by the matrix cores
            // and ran slower with that second copy of the body (FP32 at N = 1000, B = 64: 642 us
            // against 582).
            const size_t slab = (size_t)width * 16;
            const size_t base = fold_base(l, bx, c) + (size_t)lane * VEC;
            u32x4 ah[PF][NS], al[PF][NS];
            const int cnt = nq > w ? (nq - w + 3) / 4 : 0;   // slabs of this wavefront
            auto issue = [&](int d, int n) {
                int q = q0 + w + 4 * n;
                q = q < q1 ? q : q1 - 1;
                const size_t o = base + (size_t)q * slab;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    ah[d][s] = ld_a<16, NT>(reinterpret_cast<const AT*>(p.C) + o + (size_t)s * 64 * VEC);
                    if constexpr (X3) al[d][s] = ld_a<16, NT>(p.Clo + o + (size_t)s * 64 * VEC);
                }
            };
#pragma unroll
            for (int d = 0; d < PF; ++d) {
                if (FN > 1 || d < cnt) issue(d, d);
                __builtin_amdgcn_sched_barrier(0);       // slot order: slot 0 lands first
            }
            // the weights are read one slab ahead (row nq is zero)
            Acc svn[FN];
            lds_row<FN>(sl + (size_t)(w < nq ? w : nq) * NC + c16 * FN, svn);
            auto consume = [&](int d, int n) {
                Acc sv[FN];
#pragma unroll
                for (int t = 0; t < FN; ++t) sv[t] = svn[t];
                const int qn = w + 4 * (n + 1);
                lds_row<FN>(sl + (size_t)(qn < nq ? qn : nq) * NC + c16 * FN, svn);
                Acc4 Z[FN];
#pragma unroll
                for (int t = 0; t < FN; ++t) Z[t] = Acc4{0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int t = 0; t < FN; ++t) mfma_step<MKD>(Z[t], ah[d][s], al[d][s], xh[s][t], xl[s][t]);
#pragma unroll
                for (int t = 0; t < FN; ++t) Y[t] += sv[t] * Z[t];
            };
            int n0 = 0;
            for (; FN > 1 ? n0 < (nq + 3) / 4 : n0 + PF < cnt; n0 += PF) {
#pragma unroll
                for (int d = 0; d < PF; ++d) {
                    consume(d, n0 + d);
                    issue(d, n0 + PF + d);
                    // this slot's loads stay ahead of the next iterations
                    __builtin_amdgcn_sched_barrier(0x78F);
                }
            }
            if constexpr (FN == 1) {
#pragma unroll
                for (int d = 0; d < PF; ++d)
                    if (n0 + d < cnt) consume(d, n0 + d);
            }
        };
        if (width == l.kc) run(std::integral_constant<int, KW>{});
        else run(std::integral_constant<int, KW / 2>{});
    }

    // ---- add the 4 wavefront tiles in LDS (fixed order) and write the partial tile
    __syncthreads();
    Acc* red = reinterpret_cast<Acc*>(smem);             // [4][FN][4][64]
#pragma unroll
    for (int t = 0; t < FN; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((w * FN + t) * 4 + v) * 64 + lane] = Y[t][v];
    __syncthreads();
    Acc* out = reinterpret_cast<Acc*>(p.part) + (size_t)sp * p.Bpad * l.N;
    for (int e = threadIdx.x; e < 256 * FN; e += 256) {
        const int cl = e >> 4, rr = e & 15;              // local trajectory, local row
        const int t = cl % FN, cc = cl / FN;
        const int gg = MKD == MK_F64 ? (rr & 3) : (rr >> 2);
        const int v = MKD == MK_F64 ? (rr >> 2) : (rr & 3);
        const int ln = gg * 16 + cc;
        Acc sum = red[(t * 4 + v) * 64 + ln];
#pragma unroll
        for (int w2 = 1; w2 < 4; ++w2) sum += red[((w2 * FN + t) * 4 + v) * 64 + ln];
        const int row = bx * 16 + rr, b = b0 + cl;
        if (row < l.N && b < p.Bpad) out[(size_t)b * l.N + row] = sum;
    }
}

// ---------------------------------------------------------------- plan, launch

// Shapes per format: trajectories per block / 16, prefetch depth in slabs, blocks a compute
// unit holds at once (registers).  Wider tiles cost occupancy: at N = 400, B = 256 FP32 ran
// 154 us with 64 trajectories per block, 163 with 128 and 199 with 256; FP64 at B = 64 took
// 82 us with 16 or 32 and 93 with 64.
struct FoldTile { int fn, pf, cu, slab; };
constexpr int kFoldShapes = 3;
template <int DT> struct FoldTab;
template <> struct FoldTab<DT_F64> {
    static constexpr FoldTile t[kFoldShapes] = {{2, 2, 3, 1240}, {1, 2, 4, 620}, {1, 4, 3, 620}};
};
template <> struct FoldTab<DT_F32> {
    static constexpr FoldTile t[kFoldShapes] = {{4, 4, 3, 1240}, {2, 3, 4, 725}, {1, 6, 4, 390}};
};
template <> struct FoldTab<DT_BF16X3> {
    static constexpr FoldTile t[kFoldShapes] = {{4, 2, 3, 560}, {2, 3, 3, 330}, {1, 4, 4, 235}};
};

static FoldTile fold_tile(int dt, int v) {
    if (dt == DT_F64) return FoldTab<DT_F64>::t[v];
    if (dt == DT_F32) return FoldTab<DT_F32>::t[v];
    return FoldTab<DT_BF16X3>::t[v];
}

// Variants: shape v % 3; v / 3 = 0: the split of the plan below, else a fixed one of 1, 2, 3,
// 4, 6 or 8 pieces per chunk, one piece per block.
constexpr int kFoldVariants = kFoldShapes * 7;
int fold_variants() { return kFoldVariants; }

// Shape, pieces per chunk (njr) and pieces a block walks (ppb) of least estimated time.  The
// estimate is in cycles of one wavefront: a slab costs its shape's cycles times the blocks
// sharing a SIMD, or the memory latency over the ring's depth; a piece about kPiece more
// (weights, X fragments, first slabs); rounds of concurrent blocks are counted fractionally;
// and the whole is no less than the tensor's stream over HBM.  Fitted to sweeps of all shapes
// and splits at N = 64 .. 1000 and B = 7 .. 256.
FoldPlan fold_plan(int dt, const FoldLay& l, int Bpad, int variant, size_t lds_max) {
    constexpr double kPiece = 7000, kLatency = 1500;
    const size_t accb = dt == DT_F64 ? 8 : 4, per_cu = (size_t)150 << 10;
    const int gx = (l.N + 15) / 16;
    // the folded words over HBM at the measured rates (one column tile: non-temporal loads), in
    // cycles at 2.1 GHz
    const double bytes = fold_bytes(dt, l);
    const double hbm1 = bytes / 6.7e12 * 2.1e9, hbm2 = bytes / 5.7e12 * 2.1e9;
    static constexpr int kSplits[7] = {0, 1, 2, 3, 4, 6, 8};
    if (variant >= 0) variant %= kFoldVariants;
    FoldPlan pl{};
    double best = -1;
    for (int v = 0; v < kFoldShapes; ++v) {
        if (variant >= 0 && v != variant % kFoldShapes) continue;
        const FoldTile t = fold_tile(dt, v);
        const int NC = 16 * t.fn, gy = (Bpad + NC - 1) / NC;
        const size_t row = (size_t)NC * accb, red = (size_t)1024 * t.fn * accb;
        // pieces: at least what the LDS copy of the weights needs
        const int jc_max = (int)(lds_max / row) - 1;
        int njr_lo = (l.lmax + jc_max - 1) / jc_max, njr_hi = njr_lo + 7;
        if (variant >= kFoldShapes) {
            const int want = kSplits[variant / kFoldShapes];
            njr_lo = njr_hi = want > njr_lo ? want : njr_lo;
        }
        for (int njr = njr_lo; njr <= njr_hi; ++njr) {
            const int jc = (l.lmax + njr - 1) / njr, pieces = l.nk * njr;
            size_t lds = row * (jc + 1);
            if (lds < red) lds = red;
            int cu = t.cu;
            while (cu > 1 && lds * cu > per_cu) --cu;
            for (int ppb = 1; ppb <= pieces; ++ppb) {
                const int nsplit = (pieces + ppb - 1) / ppb;
                const long long blocks = (long long)gx * gy * nsplit;
                if (ppb > 1 && (blocks < 4096 || variant >= kFoldShapes)) break;
                const int share = (int)(blocks < 256LL * cu ? (blocks + 255) / 256 : cu);
                double slab = (double)t.slab * share;
                if (slab < kLatency / t.pf) slab = kLatency / t.pf;
                double rounds = (double)blocks / (256.0 * share);
                rounds = rounds <= 1 ? 1 : rounds + 0.2;  // the last blocks' tail
                double cost = rounds * ppb * ((jc + 3) / 4 * slab + kPiece);
                if (cost < (gy == 1 ? hbm1 : hbm2)) cost = gy == 1 ? hbm1 : hbm2;
                cost += nsplit + 10 * t.fn;               // equal estimates: fewer partial tiles, narrower tiles
                if (best < 0 || cost < best) {
                    best = cost;
                    pl.v = v;
                    pl.njr = njr;
                    pl.jc = jc;
                    pl.ppb = ppb;
                    pl.lds = lds;
                    pl.gy = gy;
                }
            }
        }
    }
    const int pieces = l.nk * pl.njr;
    pl.nsplit = (pieces + pl.ppb - 1) / pl.ppb;
    pl.gx = gx;
    // with one column tile nothing re-reads the tensor through L2 (FP32 at N = 700, B = 16:
    // 109 us with non-temporal loads, 128 without)
    pl.stream = pl.gy == 1 && fold_streams(dt, l);
    pl.blocks = (int)(((long long)gx * pl.gy * pl.nsplit + 7) / 8 * 8);
    return pl;
}

template <int DT, int V>
static void fold_go_v(const FoldArgs& a, const FoldPlan& pl, hipStream_t s) {
    constexpr FoldTile t = FoldTab<DT>::t[V];
    if (pl.stream) hipLaunchKernelGGL((k_fold_mm<DT, t.fn, t.pf, true>), dim3(pl.blocks), dim3(256), pl.lds, s, a);
    else hipLaunchKernelGGL((k_fold_mm<DT, t.fn, t.pf, false>), dim3(pl.blocks), dim3(256), pl.lds, s, a);
}
template <int DT>
static void fold_go(const FoldArgs& a, const FoldPlan& pl, hipStream_t s) {
    switch (pl.v) {
        case 0: fold_go_v<DT, 0>(a, pl, s); break;
        case 1: fold_go_v<DT, 1>(a, pl, s); break;
        default: fold_go_v<DT, 2>(a, pl, s); break;
    }
}

template <int DT, int V>
static hipError_t fold_attr_v(size_t lds) {
    constexpr FoldTile t = FoldTab<DT>::t[V];
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fold_mm<DT, t.fn, t.pf, true>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    const hipError_t f = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fold_mm<DT, t.fn, t.pf, false>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    return e != hipSuccess ? e : f;
}
template <int DT>
static hipError_t fold_attr(size_t lds) {
    hipError_t e = hipSuccess, q;
    if ((q = fold_attr_v<DT, 0>(lds)) != hipSuccess) e = q;
    if ((q = fold_attr_v<DT, 1>(lds)) != hipSuccess) e = q;
    if ((q = fold_attr_v<DT, 2>(lds)) != hipSuccess) e = q;
    return e;
}
hipError_t fold_set_lds_limit(size_t lds) {
    hipError_t e = hipSuccess, q;
    if ((q = fold_attr<DT_F64>(lds)) != hipSuccess) e = q;
    if ((q = fold_attr<DT_F32>(lds)) != hipSuccess) e = q;
    if ((q = fold_attr<DT_BF16X3>(lds)) != hipSuccess) e = q;
    return e;
}

void launch_fold_batched(int dt, const FoldPlan& pl0, int sp0, int nsp, const void* C, const void* Clo, const FoldLay& l,
                         int Kx, int Bpad, const void* X, const void* Xlo, const void* S, void* part, hipStream_t s) {
    FoldPlan pl = pl0;
    if (nsp != pl.nsplit) pl.blocks = (int)(((long long)pl.gx * pl.gy * nsp + 7) / 8 * 8);
    FoldArgs a{};
    a.C = C;
    a.Clo = (const unsigned short*)Clo;
    a.X = X;
    a.Xlo = (const unsigned short*)Xlo;
    a.S = S;
    a.part = part;
    a.l = l;
    a.Kx = Kx;
    a.Bpad = Bpad;
    a.njr = pl.njr;
    a.jc = pl.jc;
    a.ppb = pl.ppb;
    a.sp0 = sp0;
    a.nsplit = nsp;
    a.gx = pl.gx;
    a.gy = pl.gy;
    if (dt == DT_F64) fold_go<DT_F64>(a, pl, s);
    else if (dt == DT_F32) fold_go<DT_F32>(a, pl, s);
    else fold_go<DT_BF16X3>(a, pl, s);
}

}  // namespace rom
