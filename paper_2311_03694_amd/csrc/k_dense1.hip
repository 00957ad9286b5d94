// k_dense1.hip -- dense advection contraction for one trajectory of a large BF16 tensor (Sec.
// 2.2, eq. Cu; the 2N^3-flop term of the G-ROM; the others are in the tiled storage of kfold.h):
//     y_i = sum_j u_j * sum_k C[i][j][k] u_k,
// and, with J slabs of separate weights w, the second product of the SVD-ROM (Sec. 4.4) where
// the slabs outgrow the last-level cache (any format):
//     y_i = sum_r w_r * sum_k V[i][r][k] u_k   (w_r = sigma_r U[:,r]^T u).
//
// The tensor is stored [N][J][Np] with the k index padded by zeros to Np, a multiple
// of 8.  It is read exactly once per step, so the kernel is a stream over HBM: each row
// i of C is the contiguous (J*Np)-vector over (j, k), split into chunks with one block
// per (i, chunk).  Lanes take 16-byte non-temporal loads V elements apart, UNR
// loads in flight per lane (the first batch is issued before u is staged in LDS, to
// overlap the two latencies).  A thread walks the (j, k) plane with an incremental
// index (no division in the loop) and weights each V-vector's dot product with u by
// u_j.  BF16 pairs use the packed dot2 instruction.  Blocks write one partial sum each
// (FP32, or FP64 for the FP64 format); the BDF update adds them in a fixed order, so
// results are deterministic.  250 SVD slabs in FP32 at N = 1000: 147 us, 6.8 TB/s (tiled 149).
#include "kbody.h"

namespace rom {

template <int DT, int V, int UNR, int NT>
__global__ __launch_bounds__(NT) void k_dense_gemv(GemvJob jb) {
    dense_gemv_body<DT, V, UNR, NT>(jb, blockIdx.x);
}

static const GemvTile kGemvTiles[] = {
    {256, 4, 8192}, {256, 2, 8192}, {256, 8, 4096}, {256, 4, 16384}, {256, 4, 4096}, {256, 2, 16384},
};

int dense_gemv_variants() { return (int)(sizeof(kGemvTiles) / sizeof(kGemvTiles[0])); }
GemvTile dense_gemv_variant(int idx) {
    if (idx < 0 || idx >= dense_gemv_variants()) idx = 0;
    return kGemvTiles[idx];
}

// Number of chunks per row: about chunk_target blocks in total.
int dense_gemv_nchunk(int N, GemvTile t) {
    long long nchunk = (t.chunk_target + N - 1) / N;
    if (nchunk < 1) nchunk = 1;
    if (nchunk > 4096) nchunk = 4096;
    return (int)nchunk;
}

static long long chunk_len_of(int dt, int J, int Np, int nchunk, GemvTile t) {
    const int V = dt == DT_F64 ? 2 : dt == DT_F32 ? 4 : 8;
    const long long NN = (long long)J * Np;
    const long long step = (long long)t.threads * V;
    // a multiple of threads*V covering the row in nchunk pieces (trailing pieces may be
    // empty; their blocks write a zero partial)
    long long len = (NN + nchunk - 1) / nchunk;
    return ((len + step - 1) / step) * step;
}

GemvJob make_gemv_job(int dt, const void* C, const void* Clo, int N, int Np, int J, const void* wj,
                      const double* u_base, const long long* stepp, long long slot_stride, void* part, int nchunk,
                      GemvTile t) {
    GemvJob jb{};
    jb.C = C;
    jb.Clo = (const unsigned short*)Clo;
    jb.N = N;
    jb.Np = Np;
    jb.J = J;
    jb.wj = wj;
    jb.u_base = u_base;
    jb.stepp = stepp;
    jb.slot_stride = slot_stride;
    jb.part = part;
    jb.nchunk = nchunk;
    jb.chunk_len = chunk_len_of(dt, J, Np, nchunk, t);
    jb.blk0 = 0;
    jb.nblk = N * nchunk;
    return jb;
}

size_t dense_gemv_lds(int dt, int Np, int slabs) {
    switch (dt) {
        case DT_F64: return LdsU<DT_F64>::bytes(Np) + sizeof(double) * (size_t)slabs;
        case DT_F32: return LdsU<DT_F32>::bytes(Np) + sizeof(float) * (size_t)slabs;
        case DT_BF16: return LdsU<DT_BF16>::bytes(Np) + sizeof(float) * (size_t)slabs;
        default: return LdsU<DT_BF16X3>::bytes(Np) + sizeof(float) * (size_t)slabs;
    }
}

template <int DT>
static void gemv_go(int unr, const GemvJob& jb, hipStream_t s) {
    constexpr int V = 16 / (int)sizeof(typename Store<DT>::T);
    const size_t lds = dense_gemv_lds(DT, jb.Np, jb.wj ? jb.J : 0);
    const dim3 grid((unsigned)jb.nblk);
    if (unr == 2) hipLaunchKernelGGL((k_dense_gemv<DT, V, 2, 256>), grid, dim3(256), lds, s, jb);
    else if (unr == 8) hipLaunchKernelGGL((k_dense_gemv<DT, V, 8, 256>), grid, dim3(256), lds, s, jb);
    else hipLaunchKernelGGL((k_dense_gemv<DT, V, 4, 256>), grid, dim3(256), lds, s, jb);
}

void launch_dense_gemv(int dt, const GemvJob& jb, GemvTile t, hipStream_t s) {
    switch (dt) {
        case DT_F64: gemv_go<DT_F64>(t.unroll, jb, s); break;
        case DT_F32: gemv_go<DT_F32>(t.unroll, jb, s); break;
        case DT_BF16: gemv_go<DT_BF16>(t.unroll, jb, s); break;
        default: gemv_go<DT_BF16X3>(t.unroll, jb, s); break;
    }
}

// Staging of the slabs: a 32 x 32 patch (k, r) of a row i is read along r and written along k,
// through LDS.  Block (r patch, k patch, row).
template <int DT>
__global__ __launch_bounds__(256) void k_slab_rows(const double* __restrict__ src, int i0, int N, int R, int Np, void* dst,
                                                   unsigned short* dst_lo) {
    typedef typename Store<DT>::T T;
    __shared__ double tr[32][33];
    const int r0 = blockIdx.x * 32, k0 = blockIdx.y * 32, a = threadIdx.x % 32, q = threadIdx.x / 32;
    const double* __restrict__ Vi = src + (size_t)blockIdx.z * N * R;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = k0 + q + 8 * e;
        tr[q + 8 * e][a] = k < N && r0 + a < R ? Vi[(size_t)k * R + r0 + a] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int r = r0 + q + 8 * e, k = k0 + a;
        if (r >= R || k >= N) continue;
        const double x = tr[a][q + 8 * e];
        const size_t o = ((size_t)(i0 + blockIdx.z) * R + r) * Np + k;
        if constexpr (DT == DT_F64) {
            reinterpret_cast<T*>(dst)[o] = x;
        } else if constexpr (DT == DT_F32) {
            reinterpret_cast<T*>(dst)[o] = (float)x;
        } else {
            const float f = (float)x;
            const unsigned short h = bf16_bits(f);
            reinterpret_cast<T*>(dst)[o] = h;
            if constexpr (DT == DT_BF16X3) dst_lo[o] = bf16_bits(f - bf16_f(h));
        }
    }
}

void launch_slab_rows(int dt, const double* src, int i0, int ni, int N, int R, int Np, void* dst, void* dst_lo,
                      hipStream_t s) {
    const dim3 grid((unsigned)((R + 31) / 32), (unsigned)((N + 31) / 32), (unsigned)ni);
    unsigned short* lo = (unsigned short*)dst_lo;
    switch (dt) {
        case DT_F64: hipLaunchKernelGGL(k_slab_rows<DT_F64>, grid, dim3(256), 0, s, src, i0, N, R, Np, dst, lo); break;
        case DT_F32: hipLaunchKernelGGL(k_slab_rows<DT_F32>, grid, dim3(256), 0, s, src, i0, N, R, Np, dst, lo); break;
        case DT_BF16: hipLaunchKernelGGL(k_slab_rows<DT_BF16>, grid, dim3(256), 0, s, src, i0, N, R, Np, dst, lo); break;
        default: hipLaunchKernelGGL(k_slab_rows<DT_BF16X3>, grid, dim3(256), 0, s, src, i0, N, R, Np, dst, lo); break;
    }
}

}  // namespace rom
