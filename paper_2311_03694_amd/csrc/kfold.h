// kfold.h -- the folded dense tensor and the one-trajectory contraction of tensor slabs.
//
// C(u)u (Sec. 2.2, eq. Cu) contracts C[i][j][k] with the symmetric u_j u_k, so
//     y_i = sum_{ {j,k} } (C[i][j][k] + C[i][k][j]) u_j u_k,
// one sum of two entries per unordered pair (the entry itself for j = k): half the words
// and half the products of the unfolded form.  The sums are formed from the FP64 entries
// at staging and rounded once, so a pair carries one rounding instead of two.  (The BF16
// format rounds every entry for itself and stays unfolded.)
//
// Which of j, k is the weight and which the contracted index is free per pair.  k is cut
// into chunks of kc; chunk c contracts the j of a cyclic run of chunks ending at c itself
// (about half of them), so every chunk has the same amount of work and its j are one
// consecutive (wrapping) range.  Inside the diagonal chunk the pairs sit at k >= j, zeros
// below.  Unfolded tensors (BF16, and those whose sums would overflow the format) use the
// same storage with every chunk contracting all j, and so do the slabs of the SVD form (Sec.
// 4.4; y_i = sum_r w_r sum_k V[i][k][r] u_k) up to 200 MB, whose j is the SVD index with weights
// of its own.
//
// Storage: [row tile of 16][chunk][q = index in the chunk's j range][k / VEC][16 rows][VEC]
// (VEC = elements per 16 bytes): one lane vector of a wavefront (16 rows x 4 k-groups x 16
// bytes) is 1 KB of contiguous memory and a chunk's slabs are one contiguous run.
#pragma once

#include <type_traits>

#include "kdot.h"

namespace rom {

template <int DT> struct FoldT;
template <> struct FoldT<DT_F64> { static constexpr int KS = 8, VEC = 2, KW = 4; };
template <> struct FoldT<DT_F32> { static constexpr int KS = 16, VEC = 4, KW = 2; };
template <> struct FoldT<DT_BF16> { static constexpr int KS = 32, VEC = 8, KW = 2; };
template <> struct FoldT<DT_BF16X3> { static constexpr int KS = 32, VEC = 8, KW = 2; };

// Elements of chunk c's slabs along k: kc, or for the last chunk the 1/2 or all of it that
// holds its indices (the kernels have a copy of their loop for each).
__host__ __device__ inline int fold_width(const FoldLay& l, int c) {
    return l.N - c * l.kc <= l.kc / 2 ? l.kc / 2 : l.kc;
}

// The j range of chunk c: js, js + 1, ... (wrapping at N), len of them.
__host__ __device__ inline void fold_range(const FoldLay& l, int c, int& js, int& len) {
    if (!l.fold) {
        js = 0;
        len = l.J;
        return;
    }
    const int back = (l.nk - 1) / 2 + (l.nk % 2 == 0 && c >= l.nk / 2 ? 1 : 0);
    const int f = c - back;                              // first chunk of the run
    const int end = (c + 1) * l.kc < l.N ? (c + 1) * l.kc : l.N;
    js = (f >= 0 ? f : f + l.nk) * l.kc;
    len = f >= 0 ? end - js : end + l.N - js;
}

// Element offset of row tile `it`, chunk c (its slab q starts q * 16 * fold_width further).
__host__ __device__ inline size_t fold_base(const FoldLay& l, int it, int c) {
    return ((size_t)it * l.nk + c) * l.lmax * l.kc * 16;
}

// One trajectory: partial sums part[c * njr + jr][i] of the 16 rows of a tile over piece jr
// of chunk c's j range.  A stream over HBM: the lane keeps the u_k of its k-group in
// registers for the whole piece, so a slab costs its loads, one FMA per element and one
// weight u_j or w_j (LDS, the same for the whole wavefront).  The 4 wavefronts take every fourth
// slab (a chunk each, where all chunks run over the same j, was no faster); U slabs are in flight per wavefront, in whole rounds whose loads are not predicated
// (slabs past the end repeat the last one), so the wait is for the slot consumed only; the
// slabs left in the ring are consumed without loads behind them (a ring refilled to its end
// cost the 25 slabs of a wavefront 4 more: 100 tiled SVD slabs at N = 1000, BF16X3, 66.4 -> 63.9
// us).
// NT: non-temporal loads, for a tensor larger than the last-level cache.
template <int DT, int U, bool NT>
__device__ __forceinline__ void fold_gemv_body(const FoldJob& jb, int blk) {
    typedef typename Store<DT>::T T;
    typedef typename Store<DT>::Acc Acc;
    constexpr int KS = FoldT<DT>::KS, VEC = FoldT<DT>::VEC, KW = FoldT<DT>::KW;
    constexpr bool X3 = (DT == DT_BF16X3), BF = (DT == DT_BF16 || X3);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ Acc red[4 * 16];
    const FoldLay& l = jb.l;
    const int it = blk / (l.nk * jb.njr), rest = blk - it * (l.nk * jb.njr);
    const int c = rest / jb.njr, jr = rest - c * jb.njr;
    int js, len;
    fold_range(l, c, js, len);
    const int q0 = jr * jb.jc, q1 = q0 + jb.jc < len ? q0 + jb.jc : len;
    const int nq = q1 - q0;                              // may be <= 0: a zero partial
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int width = fold_width(l, c);
    const double* __restrict__ u = jb.u_base + (jb.stepp ? (size_t)slot_of(*jb.stepp) * jb.slot_stride : 0);
    Acc* wl = reinterpret_cast<Acc*>(smem);              // [nq] weights
    Acc acc = 0;

    auto run = [&](auto nsc) {
        constexpr int NS = decltype(nsc)::value;
        const size_t slab = (size_t)width * 16;
        const size_t base = fold_base(l, it, c) + (size_t)lane * VEC;
        const T* __restrict__ C = reinterpret_cast<const T*>(jb.C) + base;
        const unsigned short* __restrict__ Cl = X3 ? jb.Clo + base : nullptr;
        u32x4 r[U][NS], rl[U][NS];
        const int cnt = nq > w ? (nq - w + 3) / 4 : 0;   // slabs of this wavefront
        auto issue = [&](int d, int n) {
            const size_t o = (size_t)(q0 + w + 4 * (n < cnt ? n : cnt - 1)) * slab;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                r[d][s] = ld_a<16, NT>(C + o + (size_t)s * 64 * VEC);
                if constexpr (X3) rl[d][s] = ld_a<16, NT>(Cl + o + (size_t)s * 64 * VEC);
            }
        };
#pragma unroll
        for (int d = 0; d < U; ++d)
            if (d < cnt) issue(d, d);
        // the lane's u_k (fixed over the piece) and the piece's weights u_j
        Acc uf[NS][VEC];
        u32x4 uh[NS], ul[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const int k = c * l.kc + s * KS + g * VEC + v;
                uf[s][v] = (Acc)(k < l.N ? u[k] : 0.0);
            }
        if constexpr (BF) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const float f0 = uf[s][2 * p], f1 = uf[s][2 * p + 1];
                    const unsigned short h0 = bf16_bits(f0), h1 = bf16_bits(f1);
                    const unsigned short l0 = bf16_bits(f0 - bf16_f(h0)), l1 = bf16_bits(f1 - bf16_f(h1));
                    uh[s][p] = (unsigned)h0 | ((unsigned)h1 << 16);
                    ul[s][p] = (unsigned)l0 | ((unsigned)l1 << 16);
                }
        }
        for (int q = threadIdx.x; q < nq; q += 256) {
            int j = js + q0 + q;
            Acc wj;
            if (jb.wj) {
                wj = reinterpret_cast<const Acc*>(jb.wj)[j];
            } else {
                j = j < l.N ? j : j - l.N;
                wj = (Acc)u[j];
                if constexpr (DT == DT_BF16) wj = bf16_f(bf16_bits(wj));
            }
            wl[q] = wj;
        }
        __syncthreads();
        auto consume = [&](int d, int n) {
            const Acc wj = wl[w + 4 * n];
            Acc z = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if constexpr (BF) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        z = dot2_bf16(r[d][s][p], uh[s][p], z);
                        if constexpr (X3) {
                            z = dot2_bf16(r[d][s][p], ul[s][p], z);
                            z = dot2_bf16(rl[d][s][p], uh[s][p], z);
                        }
                    }
                } else {
                    Acc cv[VEC];
                    Decode<DT, VEC>::run(r[d][s], cv);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) z += cv[v] * uf[s][v];
                }
            }
            acc += wj * z;
        };
        int n0 = 0;
        for (; n0 + U < cnt; n0 += U) {
#pragma unroll
            for (int d = 0; d < U; ++d) {
                consume(d, n0 + d);
                issue(d, n0 + U + d);
            }
        }
#pragma unroll
        for (int d = 0; d < U; ++d)
            if (n0 + d < cnt) consume(d, n0 + d);
    };
    if (width == l.kc) run(std::integral_constant<int, KW>{});
    else run(std::integral_constant<int, KW / 2>{});

    // the row's 4 k-groups, then the 4 wavefronts in order
    acc += __shfl_xor(acc, 16, 64);
    acc += __shfl_xor(acc, 32, 64);
    if (lane < 16) red[w * 16 + lane] = acc;
    __syncthreads();
    if (threadIdx.x < 16) {
        const int i = it * 16 + (int)threadIdx.x;
        const Acc s = ((red[threadIdx.x] + red[16 + threadIdx.x]) + red[32 + threadIdx.x]) + red[48 + threadIdx.x];
        if (i < l.N) reinterpret_cast<Acc*>(jb.part)[(size_t)(c * jb.njr + jr) * l.N + i] = s;
    }
}

}  // namespace rom
