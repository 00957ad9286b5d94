// k_dense1.hip -- dense advection contraction for one trajectory of a large BF16 tensor (Sec.
// 2.2, eq. Cu; the 2N^3-flop term of the G-ROM; every other one is in the tiled storage of
// kfold.h):
//     y_i = sum_j u_j * sum_k C[i][j][k] u_k.
//
// The tensor is stored [N][N][Np] with the k index padded by zeros to Np, a multiple
// of 8.  It is read exactly once per step, so the kernel is a stream over HBM: each row
// i of C is the contiguous (N*Np)-vector over (j, k), split into chunks with one block
// per (i, chunk).  Lanes take 16-byte non-temporal loads V elements apart, UNR
// loads in flight per lane (the first batch is issued before u is staged in LDS, to
// overlap the two latencies).  A thread walks the (j, k) plane with an incremental
// index (no division in the loop) and weights each V-vector's dot product with u by
// u_j.  BF16 pairs use the packed dot2 instruction.  Blocks write one FP32 partial sum
// each; the BDF update adds them in a fixed order, so results are deterministic.
#include "kbody.h"

namespace rom {

template <int UNR>
__global__ __launch_bounds__(256) void k_dense_gemv(GemvJob jb) {
    dense_gemv_body<UNR>(jb, blockIdx.x);
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

static long long chunk_len_of(int N, int Np, int nchunk, GemvTile t) {
    const long long NN = (long long)N * Np;
    const long long step = (long long)t.threads * 8;
    // a multiple of one step of the block covering the row in nchunk pieces (trailing pieces
    // may be empty; their blocks write a zero partial)
    long long len = (NN + nchunk - 1) / nchunk;
    return ((len + step - 1) / step) * step;
}

GemvJob make_gemv_job(const void* C, int N, int Np, const double* u_base, const long long* stepp, long long slot_stride,
                      void* part, int nchunk, GemvTile t) {
    GemvJob jb{};
    jb.C = C;
    jb.N = N;
    jb.Np = Np;
    jb.u_base = u_base;
    jb.stepp = stepp;
    jb.slot_stride = slot_stride;
    jb.part = part;
    jb.nchunk = nchunk;
    jb.chunk_len = chunk_len_of(N, Np, nchunk, t);
    jb.blk0 = 0;
    jb.nblk = N * nchunk;
    return jb;
}

void launch_dense_gemv(const void* C, int N, int Np, const double* u_base, const long long* stepp, long long slot_stride,
                       void* part, int nchunk, GemvTile t, hipStream_t s) {
    const GemvJob jb = make_gemv_job(C, N, Np, u_base, stepp, slot_stride, part, nchunk, t);
    const size_t lds = LdsU<DT_BF16>::bytes(Np);
    const dim3 grid((unsigned)jb.nblk);
    if (t.unroll == 2) hipLaunchKernelGGL((k_dense_gemv<2>), grid, dim3(256), lds, s, jb);
    else if (t.unroll == 8) hipLaunchKernelGGL((k_dense_gemv<8>), grid, dim3(256), lds, s, jb);
    else hipLaunchKernelGGL((k_dense_gemv<4>), grid, dim3(256), lds, s, jb);
}

}  // namespace rom
