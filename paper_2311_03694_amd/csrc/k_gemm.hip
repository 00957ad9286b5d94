// k_gemm.hip -- skinny products of the batched path on the matrix cores:
//   Y[b][m] = sum_k A[m][k] X[b][k]     (M rows, K contracted, Bpad <= a few hundred columns)
// used for the CP projections [Bf|Cf]^T u and the CP scatter Af W (Sec. 3.1, eq. tc_ap)
// and for the batched Helmholtz apply Hinv_k rhs (eq. nse_d1, dense stiffness).
//
// Block = NW wavefronts over one 16-row tile of A and 16*FN columns, over the whole of K:
// wavefront w takes the w-th part of the K steps (one step = one 16-byte lane vector per
// lane: 32 k in BF16, 16 in FP32, 8 in FP64) and streams its A and X fragments through a
// PF-deep register ring; the NW partial tiles are added in LDS in a fixed order and written
// straight to Y (no partial buffers, no second pass).  With one block per output tile the
// grid is ceil(M/16) x (column tiles), which fills the device for the shapes of this path; A
// is read once per column tile (column tiles of one row tile run next to each other on one
// XCD and share its L2).
//
// The products of a step read A, X and W in tiles (TL; tile_off, kcommon.h): a fragment is
// 1 KB of contiguous memory.  In rows it was 16 pieces of 64 bytes, at which a compute unit
// took in about 20 bytes a cycle: N = 1000, R = 2000, B = 64 FP32 33 us per step, in tiles
// 24.  A wavefront issues no fragment past its last step: with a ring refilled to its end,
// the 2 to 8 steps a wavefront has in small products cost as many again (N = 100, R = 150,
// B = 12: 9.8 -> 7.0 us per step).
//
// Epilogues (EPI):
//  * PLAIN writes Y.
//  * PAIR (the CP projections): a block takes row tile r of Bf^T and the same tile of
//    Cf^T (rows pair_off apart), so it holds s[b][r] and t[b][r] together and writes the
//    Hadamard product W[b][r] = lam_r s t (eq. tc_ap) instead of the projections.
//  * UPDATE / RHS (the CP scatter of a step): each output y^n[b][i] goes straight into
//    the BDFk/EXTk right-hand side of eq. nse_d1; UPDATE (diagonal stiffness) also
//    solves for u^{n+1}, stores it and leaves the energy of its 16 rows per trajectory,
//    and one extra block closes the previous level and advances the step counter (this
//    kernel is then the step's update kernel); RHS stores the right-hand side for the
//    Helmholtz apply.
//  * FINISH (the batched Helmholtz apply of a step): the outputs are u^{n+1}; they are
//    stored with their energy partials, and one extra block closes the step.
//  * SKEW (the CP projections of factors with skew column pairs, Sec. 3.3): A is the pair
//    form [P + R][Np] (the P distinct columns of Bf, then the columns of Af); a block
//    takes 16 pairs, each lane three rows (beta, alpha, gamma of its pair), and writes
//    W[b][c0] = lam beta gamma and W[b][c1] = -lam beta alpha; pairs past P write the
//    zero padding of W.
#include "als.h"
#include "kmfma.h"
#include "kstep.h"

namespace rom {

struct GemmArgs {
    const void* A;                 // [M][lda] rows in the operator's storage format, or tiled
    const unsigned short* Alo;     // BF16X3 low words of A
    const void* X;                 // [Bpad][ldx] in the MFMA operand format, or tiled
    const unsigned short* Xlo;     // BF16X3 low words of X
    void* Y;                       // [Bpad][M] (accumulation type); PAIR, SKEW: W, tiled
    int M, K, Bpad;
    long long lda, ldx;            // rows only
    int gx, gy;                    // row tiles, column tiles
    int ksplit;                    // PLAIN: K ranges, one partial product each (Y + split * M * Bpad)
    int bstore;                    // PLAIN: columns b of Y stored (0: all Bpad)
    const long long* kstep;        // non-null: set (BDF order at *kstep - 1) of A
    long long set;                 // tiled: elements of one set of A
    const void* lam;               // PAIR, SKEW: lam (accumulation type)
    int skew_P, skew_layout;       // SKEW: pairs, layout (1 interleaved, 2 blocked)
    int wkt;                       // PAIR, SKEW: row length of W (whole steps of its product)
    StepArgs st;                   // UPDATE, RHS: the state of the step (M = N rows)
};

enum { EPI_PLAIN = 0, EPI_PAIR = 1, EPI_UPDATE = 2, EPI_RHS = 3, EPI_FINISH = 4, EPI_SKEW = 5 };

template <int ADT, int MKD, int FN, int PF, int EPI, bool TL>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs p) {
    constexpr int NW = 4;                                // wavefronts
    constexpr bool PAIR = (EPI == EPI_PAIR);
    constexpr bool SKEW = (EPI == EPI_SKEW);
    constexpr bool CLOSE = (EPI == EPI_UPDATE || EPI == EPI_FINISH);   // writes level n+1
    typedef MfmaT<MKD> Tr;
    typedef typename Tr::X XT;
    typedef typename Tr::Acc Acc;
    typedef typename Tr::Acc4 Acc4;
    constexpr int KS = Tr::KS, VEC = Tr::VEC;
    constexpr bool X3 = (MKD == MK_BF16X3);
    // a FP32 product over BF16 words (the CP scatter of the BF16 formats) reads 4 words
    // per lane vector and converts them when the slot is consumed, not when it is
    // loaded (a conversion at load time would wait for the load right away)
    constexpr bool CVT = (MKD == MK_F32 && ADT != DT_F32);
    constexpr int AV = CVT ? 4 : (int)(16 / sizeof(typename Store<ADT>::T));
    static_assert(AV == VEC, "lane vectors of A and X must cover the same k");
    constexpr int NA = PAIR ? 2 : SKEW ? 3 : 1;          // A rows per lane (row and partner(s))
    extern __shared__ __attribute__((aligned(16))) char smem[];
    Acc* red = reinterpret_cast<Acc*>(smem);             // [NA][NW][FN][4][64]

    const int nks = EPI == EPI_PLAIN ? p.ksplit : 1;
    const int nwork = p.gx * p.gy * nks + (CLOSE ? 1 : 0);
    const int per = (nwork + 7) / 8;
    const int wi = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (wi >= nwork) return;
    if constexpr (CLOSE) {
        if (wi == nwork - 1) {                           // the step-closing block
            close_and_advance(p.st, *p.st.step, p.gx);
            return;
        }
    }
    // the K ranges of one tile are consecutive work items (one XCD, shared X rows)
    const int ks = wi % nks, tile = wi / nks;
    const int by = tile % p.gy, bx = tile / p.gy;

    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rowbase = bx * 16, b0 = by * 16 * FN;
    // this block's K steps [kb, kb + kn), split over the NW wavefronts
    const int ksteps_all = (p.K + KS - 1) / KS;
    const int kper = (ksteps_all + nks - 1) / nks;
    const int kb = ks * kper;
    const int ksteps = kb < ksteps_all ? (ksteps_all - kb < kper ? ksteps_all - kb : kper) : 0;
    const int wsb = ksteps / NW, wse = ksteps - wsb * NW;
    const int ns = wsb + (w < wse ? 1 : 0);
    const int s0 = kb + w * wsb + (w < wse ? w : wse);

    // Tiled: fragment (row tile, step) at ((tile * steps + step) * 16 KS + lane * VEC.  Rows:
    // the lane's row (rows past M are clamped for loads and never stored) and columns.
    const size_t kbase = TL && p.kstep ? (size_t)(bdf_order(*p.kstep) - 1) * p.set : 0;
    size_t arow[NA], xrow[FN];
    if constexpr (TL) {
#pragma unroll
        for (int h = 0; h < NA; ++h)
            arow[h] = kbase + h * (size_t)p.set + (size_t)bx * ksteps_all * 16 * KS + (size_t)lane * VEC;
#pragma unroll
        for (int t = 0; t < FN; ++t) xrow[t] = (size_t)(by * FN + t) * ksteps_all * 16 * KS + (size_t)lane * VEC;
    } else {
        int r = rowbase + c16;
        r = r < p.M ? r : p.M - 1;
        arow[0] = (size_t)r * p.lda;
#pragma unroll
        for (int t = 0; t < FN; ++t) {
            int b = b0 + t * 16 + c16;
            b = b < p.Bpad ? b : p.Bpad - 1;
            xrow[t] = (size_t)b * p.ldx;
        }
    }

    Acc4 Z[NA][FN];
#pragma unroll
    for (int h = 0; h < NA; ++h)
#pragma unroll
        for (int t = 0; t < FN; ++t) Z[h][t] = Acc4{0, 0, 0, 0};

    // Ring of PF steps: whole rounds of PF steps that refill the slots they consume (steps
    // past the last one repeat it), then the 1 .. PF steps left in the ring.  The rounds have
    // no branches and wait only for the slot they use.  Rows: addresses past K are clamped to
    // the last lane vector of the row and their X fragments selected to zero when consumed
    // (tiles are padded with zeros).
    u32x4 ah[NA][PF], al[NA][PF], xh[PF][FN], xl[PF][FN];
    int kq[PF];
    auto issue = [&](int d, int q) {
        const int st = s0 + (q < ns ? q : ns - 1);
        int k = TL ? st * 16 * KS : st * KS + g * VEC;
        if constexpr (!TL) {
            kq[d] = k;
            k = k < p.K ? k : p.K - VEC;
        }
#pragma unroll
        for (int h2 = 0; h2 < NA; ++h2) {
            const size_t ar = arow[h2];
            if constexpr (CVT) {
                const u32x2 h = ld_plain<8>(reinterpret_cast<const unsigned short*>(p.A) + ar + k);
                u32x2 l = u32x2{0u, 0u};
                if constexpr (ADT == DT_BF16X3) l = ld_plain<8>(p.Alo + ar + k);
                ah[h2][d] = u32x4{h[0], h[1], l[0], l[1]};
            } else {
                load_a<ADT, MKD, false>(p.A, p.Alo, ar + k, ah[h2][d], al[h2][d]);
            }
        }
#pragma unroll
        for (int t = 0; t < FN; ++t) {
            xh[d][t] = ld_plain<16>(reinterpret_cast<const XT*>(p.X) + xrow[t] + k);
            if constexpr (X3) xl[d][t] = ld_plain<16>(p.Xlo + xrow[t] + k);
            else xl[d][t] = u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto consume = [&](int d) {
        const bool live = TL || kq[d] < p.K;
        const u32x4 z = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int h2 = 0; h2 < NA; ++h2) {
            u32x4 av = ah[h2][d];
            if constexpr (CVT) {
                // 4 BF16 words (plus their low words) -> 4 FP32 values, hi + lo exact
                float f[4] = {bf16_lo_f(av[0]), bf16_hi_f(av[0]), bf16_lo_f(av[1]), bf16_hi_f(av[1])};
                if constexpr (ADT == DT_BF16X3) {
                    f[0] += bf16_lo_f(av[2]);
                    f[1] += bf16_hi_f(av[2]);
                    f[2] += bf16_lo_f(av[3]);
                    f[3] += bf16_hi_f(av[3]);
                }
                av = u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
            }
#pragma unroll
            for (int t = 0; t < FN; ++t) {
                const u32x4 xv = live ? xh[d][t] : z;
                const u32x4 xlv = live ? xl[d][t] : z;
                mfma_step<MKD>(Z[h2][t], av, al[h2][d], xv, xlv);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < PF; ++d) {
        if (d < ns) issue(d, d);
        __builtin_amdgcn_sched_barrier(0);               // slot order: slot 0 lands first
    }
    // the step's level, and the history of the outputs this thread finishes (behind the ring's
    // loads, so their latency is the same one)
    const long long n = EPI >= EPI_UPDATE ? *p.st.step : 0;
    constexpr bool STEP = (EPI == EPI_UPDATE || EPI == EPI_RHS);
    constexpr int OUTS = (4 * FN + NW - 1) / NW;         // outputs per thread
    constexpr bool EARLY = STEP && OUTS <= 2;
    BdfHist hist[EARLY ? OUTS : 1];
    double hd[EARLY ? OUTS : 1];
    if constexpr (EARLY) {
#pragma unroll
        for (int o = 0; o < OUTS; ++o) {
            const int e = (int)threadIdx.x + o * 64 * NW, row = rowbase + (e & 15), b = b0 + (e >> 4);
            if (e < 256 * FN && row < p.M && b < p.st.B) {
                hist[o] = bdf_hist_point(p.st, n, bdf_order(n), b, row);
                if constexpr (EPI == EPI_UPDATE) hd[o] = p.st.hdiag[(size_t)(bdf_order(n) - 1) * p.st.N + row];
            }
        }
    }
    int q0 = 0;
    for (; q0 + PF < ns; q0 += PF) {
#pragma unroll
        for (int d = 0; d < PF; ++d) {
            consume(d);
            issue(d, q0 + PF + d);
            // nothing crosses: later slots' arithmetic hoisted above these loads
            // would push the loads to the end of the body and defeat the ring
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < PF; ++d)
        if (q0 + d < ns) consume(d);

    // ---- add the NW wavefront tiles (fixed order) and write Y (PAIR: W = lam s t)
    constexpr int RS = NW * FN * 4 * 64;                 // one A row set of red
#pragma unroll
    for (int h = 0; h < NA; ++h)
#pragma unroll
        for (int t = 0; t < FN; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[h * RS + ((w * FN + t) * 4 + v) * 64 + lane] = Z[h][t][v];
    __syncthreads();
    Acc* out = reinterpret_cast<Acc*>(p.Y) + (size_t)ks * p.M * p.Bpad;
#pragma unroll
    for (int o = 0; o < OUTS; ++o) {
        const int e = (int)threadIdx.x + o * 64 * NW;
        if (256 * FN % (64 * NW) != 0 && e >= 256 * FN) break;
        const int cl = e >> 4, rr = e & 15;              // local column, local row
        const int t = cl >> 4, cc = cl & 15;
        const int gg = MKD == MK_F64 ? (rr & 3) : (rr >> 2);
        const int v = MKD == MK_F64 ? (rr >> 2) : (rr & 3);
        const int ln = gg * 16 + cc;
        Acc sum[NA];
#pragma unroll
        for (int h = 0; h < NA; ++h) {
            sum[h] = red[h * RS + (t * 4 + v) * 64 + ln];
#pragma unroll
            for (int w2 = 1; w2 < NW; ++w2) sum[h] += red[h * RS + ((w2 * FN + t) * 4 + v) * 64 + ln];
        }
        const int row = rowbase + rr, b = b0 + cl;
        if constexpr (SKEW) {
            if (b < p.Bpad) {
                constexpr int WKS = sizeof(Acc) == 8 ? 8 : 16, WV = 16 / (int)sizeof(Acc);
                auto w_at = [&](int r2) -> Acc& { return out[tile_off<WKS, WV>(p.wkt, b, r2)]; };
                if (row < p.skew_P) {
                    const int c0 = p.skew_layout == 1 ? 2 * row : row;
                    const int c1 = p.skew_layout == 1 ? 2 * row + 1 : p.skew_P + row;
                    const Acc* lam = reinterpret_cast<const Acc*>(p.lam);
                    w_at(c0) = lam[c0] * sum[0] * sum[2];
                    w_at(c1) = lam[c1] * sum[0] * (-sum[1]);
                } else {
                    const int r2 = 2 * row;                       // zero padding of W past R = 2P
                    if (r2 < p.wkt) w_at(r2) = 0;
                    if (r2 + 1 < p.wkt) w_at(r2 + 1) = 0;
                }
            }
        } else if constexpr (PAIR) {
            constexpr int WKS = sizeof(Acc) == 8 ? 8 : 16, WV = 16 / (int)sizeof(Acc);
            if (row < p.wkt && b < p.Bpad)
                out[tile_off<WKS, WV>(p.wkt, b, row)] =
                    row < p.M ? reinterpret_cast<const Acc*>(p.lam)[row] * sum[0] * sum[1] : 0;
        } else if constexpr (EPI == EPI_PLAIN) {
            if (row < p.M && b < (p.bstore > 0 ? p.bstore : p.Bpad)) out[(size_t)b * p.M + row] = sum[0];
        } else {
            const StepArgs& a = p.st;
            double ev = 0.0;
            if (row < p.M && b < a.B) {
                if constexpr (EPI == EPI_FINISH) {
                    const double un = (double)sum[0];
                    write_level(a, n + 1, b, row, un);
                    ev = un * un;
                } else {
                    const int k = bdf_order(n);
                    const BdfCoef c = bdf_coef(k);
                    double rhs;
                    if constexpr (EARLY) rhs = bdf_rhs_hist(a, n, c, k, b, row, (double)sum[0], hist[o]);
                    else rhs = bdf_rhs_point(a, n, c, k, b, row, (double)sum[0]);
                    if constexpr (EPI == EPI_UPDATE) {
                        double h = 0.0;
                        if constexpr (EARLY) h = hd[o];
                        else h = a.hdiag[(size_t)(k - 1) * a.N + row];
                        const double un = rhs * h;
                        write_level(a, n + 1, b, row, un);
                        ev = un * un;
                    } else {
                        a.rhs[tile_off<8, 2>(a.Np, b, row)] = rhs;
                    }
                }
            }
            if constexpr (CLOSE) {
                // the tile's 16 rows of trajectory b sit in 16 consecutive lanes
                ev += __shfl_xor(ev, 8, 16);
                ev += __shfl_xor(ev, 4, 16);
                ev += __shfl_xor(ev, 2, 16);
                ev += __shfl_xor(ev, 1, 16);
                if (rr == 0 && b < a.B) epart_of(a, n + 1)[(size_t)b * a.enmax + bx] = ev;
            }
        }
    }
}

// ---------------------------------------------------------------- planning, launch

// Column-tile width: 1, 2, 3 force FN = 1, 2, 4; 0 (row-major operands) picks the widest that
// still gives about one block per compute unit.  The tiled step products take FN = 1 unless a
// caller's knob (0 .. 3) says otherwise: in every format and at every size measured, more blocks and
// waves were worth more than re-using a fragment of A (N = 1000, R = 2000, B = 64 FP32: 22.4,
// 27.6 and 44 us per step with FN = 1, 2, 4).  So were 4 wavefronts per block against 8 or 16
// (22.5, 23.2, 25.9 us) and a ring of 8 steps against 6, 12 or 16.
constexpr int kGemmVariants = 4;
int gemm_variants() { return kGemmVariants; }

static int gemm_fn(int M, int Bpad, int v) {
    const int nct = Bpad / 16;
    if (v == 1) return 1;
    if (v == 2) return nct % 2 == 0 ? 2 : 1;
    if (v == 3) return nct % 4 == 0 ? 4 : (nct % 2 == 0 ? 2 : 1);
    // widest tile that still gives about one block per CU
    const int gx = (M + 15) / 16;
    for (int fn : {4, 2})
        if (nct % fn == 0 && (long long)gx * (nct / fn) >= 224) return fn;
    return 1;
}

GemmPlan gemm_plan(int M, int Bpad, int variant) {
    GemmPlan pl{};
    pl.fn = gemm_fn(M, Bpad, variant < 0 ? 0 : variant);
    pl.gx = (M + 15) / 16;
    pl.gy = Bpad / (16 * pl.fn);
    pl.blocks = (pl.gx * pl.gy + 7) / 8 * 8;
    pl.ksplit = 1;
    return pl;
}

// The widest column tiles (each A fragment feeds up to four MFMA tiles; with one 16-column
// tile a block's loads run at the compute unit's vector-load rate), then K ranges where
// the output tiles leave compute units idle: about one block per compute unit (about two
// were slower: more prologues and reductions), each wavefront keeping at least 4 K steps
// (8 FP64 values a step), at most 8 ranges.  N = 1000, B = 64, K = 2000: 17.5 -> 14.0 us.
GemmPlan gemm_plan_splitk(int M, int K, int Bpad) {
    GemmPlan pl = gemm_plan(M, Bpad, 3);
    const int tiles = pl.gx * pl.gy, ksteps = (K + 7) / 8;
    int ks = 256 / tiles;
    ks = ks < 1 ? 1 : ks > 8 ? 8 : ks;
    while (ks > 1 && ksteps / ks < 16) --ks;
    pl.ksplit = ks;
    pl.blocks = (tiles * ks + 7) / 8 * 8;
    return pl;
}

template <int ADT, int MKD, int FN, int PF, int EPI, bool TL>
static void gemm_launch(const GemmArgs& a, const GemmPlan& pl, hipStream_t s) {
    constexpr int NA = EPI == EPI_PAIR ? 2 : EPI == EPI_SKEW ? 3 : 1;
    const size_t lds = (size_t)NA * 4 * FN * 256 * sizeof(typename MfmaT<MKD>::Acc);
    hipLaunchKernelGGL((k_gemm<ADT, MKD, FN, PF, EPI, TL>), dim3(pl.blocks), dim3(256), lds, s, a);
}

template <int ADT, int MKD, int EPI = EPI_PLAIN, bool TL = true>
static void gemm_go(const GemmArgs& a, const GemmPlan& pl, hipStream_t s) {
    if (pl.fn == 4) gemm_launch<ADT, MKD, 4, 4, EPI, TL>(a, pl, s);
    else if (pl.fn == 2) gemm_launch<ADT, MKD, 2, 6, EPI, TL>(a, pl, s);
    else gemm_launch<ADT, MKD, 1, 8, EPI, TL>(a, pl, s);
}

static GemmArgs gemm_args(const GemmPlan& pl, const void* A, const void* Alo, const void* X, const void* Xlo, void* Y,
                          int M, int K, int Bpad) {
    GemmArgs a{};
    a.A = A;
    a.Alo = (const unsigned short*)Alo;
    a.X = X;
    a.Xlo = (const unsigned short*)Xlo;
    a.Y = Y;
    a.M = M;
    a.K = K;
    a.Bpad = Bpad;
    a.gx = pl.gx;
    a.gy = pl.gy;
    a.ksplit = pl.ksplit > 0 ? pl.ksplit : 1;
    return a;
}

// ---------------------------------------------------------------- operand tiles

static int gemm_ks(int dt) { return dt == DT_F64 ? 8 : dt == DT_F32 ? 16 : 32; }
int gemm_kt(int dt, int K) { return (K + gemm_ks(dt) - 1) / gemm_ks(dt) * gemm_ks(dt); }
size_t gemm_tiled_elems(int sdt, int rows, int K) { return (size_t)((rows + 15) / 16 * 16) * gemm_kt(sdt, K); }

struct TileRows { int r0[3], rmul[3]; };
// Set blockIdx.z, one thread per lane vector of the tiled copy: rows r0 + rmul * row of src.
template <class T, int KS, int VEC>
__global__ void k_gemm_tile(const T* __restrict__ src, T* __restrict__ dst, int rows, int K, long long ld, int steps,
                            long long units, TileRows tr) {
    const int set = blockIdx.z;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < units; q += (long long)gridDim.x * blockDim.x) {
        const int r = (int)(q & 15), g = (int)(q >> 4) & 3;
        const long long rest = q >> 6;
        const int step = (int)(rest % steps);
        const long long row = (rest / steps) * 16 + r;
        const int k0 = step * KS + g * VEC;
        T v[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            v[e] = row < rows && k0 + e < K ? src[(tr.r0[set] + tr.rmul[set] * row) * ld + k0 + e] : (T)0;
        T* d = dst + ((size_t)set * units + q) * VEC;
#pragma unroll
        for (int e = 0; e < VEC; ++e) d[e] = v[e];
    }
}

void launch_gemm_tile(int eb, int sdt, const void* src, void* dst, int rows, int K, long long ld, int sets, const int* r0,
                      const int* rmul, hipStream_t s) {
    TileRows tr{};
    for (int q = 0; q < sets && q < 3; ++q) {
        tr.r0[q] = r0[q];
        tr.rmul[q] = rmul[q];
    }
    const int steps = gemm_kt(sdt, K) / gemm_ks(sdt);
    const long long units = (long long)((rows + 15) / 16) * steps * 64;
    const long long want = (units + 255) / 256;
    const dim3 grid((unsigned)(want < 4096 ? want : 4096), 1, (unsigned)sets);
    if (eb == 8)
        hipLaunchKernelGGL((k_gemm_tile<double, 8, 2>), grid, dim3(256), 0, s, (const double*)src, (double*)dst, rows, K, ld,
                           steps, units, tr);
    else if (eb == 4)
        hipLaunchKernelGGL((k_gemm_tile<float, 16, 4>), grid, dim3(256), 0, s, (const float*)src, (float*)dst, rows, K, ld,
                           steps, units, tr);
    else if (sdt == DT_F32)
        hipLaunchKernelGGL((k_gemm_tile<unsigned short, 16, 4>), grid, dim3(256), 0, s, (const unsigned short*)src,
                           (unsigned short*)dst, rows, K, ld, steps, units, tr);
    else
        hipLaunchKernelGGL((k_gemm_tile<unsigned short, 32, 8>), grid, dim3(256), 0, s, (const unsigned short*)src,
                           (unsigned short*)dst, rows, K, ld, steps, units, tr);
}

// ---------------------------------------------------------------- the products

// CP projections and their Hadamard product in one pass: W[b][r] = lam_r (Bf^T u_b)_r
// (Cf^T u_b)_r over the tiled sets Bf^T and Cf^T; W in the accumulation type, tiled.  The
// plan's column-tile width is kept, its row tiles are those of Rp rows.
void launch_gemm_proj_pair(int dt, const GemmPlan& pl0, const void* BCt, const void* BCt_lo, int Np, int Rp, int Bpad,
                           const void* X, const void* Xlo, const void* lam, void* W, hipStream_t s) {
    GemmPlan pl = pl0;
    pl.gx = (Rp + 15) / 16;
    pl.gy = Bpad / (16 * pl.fn);
    pl.blocks = (pl.gx * pl.gy + 7) / 8 * 8;
    GemmArgs a = gemm_args(pl, BCt, BCt_lo, X, Xlo, W, Rp, Np, Bpad);
    a.set = (long long)gemm_tiled_elems(dt, Rp, Np);
    a.wkt = gemm_kt(dt == DT_F64 ? DT_F64 : DT_F32, Rp);
    a.lam = lam;
    switch (dt) {
        case DT_F64: gemm_go<DT_F64, MK_F64, EPI_PAIR>(a, pl, s); break;
        case DT_F32: gemm_go<DT_F32, MK_F32, EPI_PAIR>(a, pl, s); break;
        case DT_BF16: gemm_go<DT_BF16, MK_BF16, EPI_PAIR>(a, pl, s); break;
        default: gemm_go<DT_BF16X3, MK_BF16X3, EPI_PAIR>(a, pl, s); break;
    }
}

// CP projections of factors with skew column pairs and their Hadamard product, from the
// pair form's tiled sets (SKEW epilogue): W in the accumulation type, tiled.
void launch_gemm_proj_skew(int dt, const GemmPlan& pl0, const void* SK, const void* SK_lo, int Np, int P, int layout,
                           int Rp, int Bpad, const void* X, const void* Xlo, const void* lam, void* W, hipStream_t s) {
    GemmPlan pl = pl0;
    pl.gx = (Rp / 2 + 15) / 16;
    pl.gy = Bpad / (16 * pl.fn);
    pl.blocks = (pl.gx * pl.gy + 7) / 8 * 8;
    GemmArgs a = gemm_args(pl, SK, SK_lo, X, Xlo, W, P, Np, Bpad);
    // row tiles past the pairs (the padding of W) read the sets' last tile instead
    a.set = (long long)gemm_tiled_elems(dt, Rp / 2, Np);
    a.skew_P = P;
    a.skew_layout = layout;
    a.wkt = gemm_kt(dt == DT_F64 ? DT_F64 : DT_F32, Rp);
    a.lam = lam;
    switch (dt) {
        case DT_F64: gemm_go<DT_F64, MK_F64, EPI_SKEW>(a, pl, s); break;
        case DT_F32: gemm_go<DT_F32, MK_F32, EPI_SKEW>(a, pl, s); break;
        case DT_BF16: gemm_go<DT_BF16, MK_BF16, EPI_SKEW>(a, pl, s); break;
        default: gemm_go<DT_BF16X3, MK_BF16X3, EPI_SKEW>(a, pl, s); break;
    }
}

// CP scatter: Y[b][i] = sum_r Af[i][r] W[b][r] (Af and W tiled), W in FP32 (FP64 for DT_F64);
// the BF16 formats contract their factor words with FP32 MFMA.
void launch_gemm_scatter(int dt, const GemmPlan& pl, const void* Af, const void* Af_lo, int N, int Rp, int Bpad,
                         const void* W, void* Y, hipStream_t s) {
    const GemmArgs a = gemm_args(pl, Af, Af_lo, W, nullptr, Y, N, Rp, Bpad);
    switch (dt) {
        case DT_F64: gemm_go<DT_F64, MK_F64>(a, pl, s); break;
        case DT_F32: gemm_go<DT_F32, MK_F32>(a, pl, s); break;
        case DT_BF16: gemm_go<DT_BF16, MK_F32>(a, pl, s); break;
        default: gemm_go<DT_BF16X3, MK_F32>(a, pl, s); break;
    }
}

// CP scatter of a step: y^n = Af W goes straight into the BDF right-hand side; with a
// diagonal stiffness (diag = 1) the kernel also solves for u^{n+1} and closes the step
// (one extra block), else it stores the right-hand side for the Helmholtz apply.
void launch_gemm_scatter_step(int dt, const GemmPlan& pl0, const void* Af, const void* Af_lo, int N, int Rp,
                              int Bpad, const void* W, const StepArgs& st, int diag, hipStream_t s) {
    GemmPlan pl = pl0;
    if (diag) pl.blocks = (pl.gx * pl.gy + 1 + 7) / 8 * 8;
    GemmArgs a = gemm_args(pl, Af, Af_lo, W, nullptr, nullptr, N, Rp, Bpad);
    a.st = st;
    if (diag) {
        switch (dt) {
            case DT_F64: gemm_go<DT_F64, MK_F64, EPI_UPDATE>(a, pl, s); break;
            case DT_F32: gemm_go<DT_F32, MK_F32, EPI_UPDATE>(a, pl, s); break;
            case DT_BF16: gemm_go<DT_BF16, MK_F32, EPI_UPDATE>(a, pl, s); break;
            default: gemm_go<DT_BF16X3, MK_F32, EPI_UPDATE>(a, pl, s); break;
        }
    } else {
        switch (dt) {
            case DT_F64: gemm_go<DT_F64, MK_F64, EPI_RHS>(a, pl, s); break;
            case DT_F32: gemm_go<DT_F32, MK_F32, EPI_RHS>(a, pl, s); break;
            case DT_BF16: gemm_go<DT_BF16, MK_F32, EPI_RHS>(a, pl, s); break;
            default: gemm_go<DT_BF16X3, MK_F32, EPI_RHS>(a, pl, s); break;
        }
    }
}

// Plain FP64 product of row-major operands Y[b][m] = sum_k A[m][k] X[b][k] (setup work, the
// full form's terms).
void launch_gemm_f64(const GemmPlan& pl, const double* A, long long lda, const double* X, long long ldx, double* Y,
                     int M, int K, int Bpad, hipStream_t s) {
    GemmArgs a = gemm_args(pl, A, nullptr, X, nullptr, Y, M, K, Bpad);
    a.lda = lda;
    a.ldx = ldx;
    gemm_go<DT_F64, MK_F64, EPI_PLAIN, false>(a, pl, s);
}

void launch_gemm_f64_rows(const GemmPlan& pl, const double* A, long long lda, const double* X, long long ldx,
                          double* Y, int M, int K, int Bpad, int rows, hipStream_t s) {
    GemmArgs a = gemm_args(pl, A, nullptr, X, nullptr, Y, M, K, Bpad);
    a.lda = lda;
    a.ldx = ldx;
    a.bstore = rows;
    gemm_go<DT_F64, MK_F64, EPI_PLAIN, false>(a, pl, s);
}

// Batched Helmholtz apply of a step: u^{n+1}[b][i] = sum_m Hinv_k[i][m] rhs[b][m] (FP64, both
// tiled), k from the device step counter, stored into the state with its energy partials; one
// extra block closes the step.
void launch_gemm_helm(const GemmPlan& pl0, const double* hinv, int N, int Np, int Bpad, const double* rhs,
                      const long long* stepp, const StepArgs& st, hipStream_t s) {
    GemmPlan pl = pl0;
    pl.blocks = (pl.gx * pl.gy + 1 + 7) / 8 * 8;
    GemmArgs a = gemm_args(pl, hinv, nullptr, rhs, nullptr, nullptr, N, Np, Bpad);
    a.kstep = stepp;
    a.set = (long long)gemm_tiled_elems(DT_F64, N, Np);
    a.st = st;
    gemm_go<DT_F64, MK_F64, EPI_FINISH>(a, pl, s);
}

}  // namespace rom
