// What the two fp32 contraction kernels (gemm_f32.hip: fp32 MFMAs; gemm_f32x3.hip: bf16 MFMAs on three terms per value)
// have in common.
#pragma once
#include "device.h"
#include "kernels.h"

namespace sfb {

struct GemmF32Params {
    const float* A;
    const float* B;
    float* C;
    const float* aux;
    const float* L_ptr;
    int64_t lda, ldb, ldc;
    int64_t M, N, K;
    float eta, lambda;
    int tiles_m, tiles_n;
    int split_k;          // > 1: workgroup z of a tile covers k-slices [z * per_split, (z + 1) * per_split) and writes partial[z]
    int64_t per_split;    // k-slices per split
    float* partial;       // [split_k][M][N]
    int* parts;           // (host) GemmF32Args::parts
    int num_xcd;
    int group_m;          // raster: groups of group_m row-tiles, row-tile index fastest inside a group
};

template <int EPI>
__device__ __forceinline__ float gemm_combine(float old, float acc, float eta, float invL, float th)
{
    if (EPI == EPI_RMW) return old - eta * acc;
    if (EPI == EPI_RESID) return old - acc;
    if (EPI == EPI_SHRINK) {
        const float t = old + acc * invL;
        return t > th ? t - th : (t < -th ? t + th : 0.f);
    }
    return acc;
}

// Row and column tile of a workgroup: each XCD (one L2) takes a contiguous range of a raster in which consecutive tiles
// form compact blocks (group_m row-tiles x as many column-tiles): the workgroups of an XCD walk k together, so a line of
// an operand panel is fetched into that L2 once and found there by the other tiles that share the panel.
__device__ __forceinline__ void gemm_tile_of(const GemmF32Params& p, uint32_t& tile_m, uint32_t& tile_n)
{
    // (32-bit: a 64-bit division is some hundred instructions in front of the first load)
    const uint32_t tiles = gridDim.x, xcds = (uint32_t)p.num_xcd, tiles_n = (uint32_t)p.tiles_n, tiles_m = (uint32_t)p.tiles_m;
    const uint32_t x = blockIdx.x % xcds, wi = blockIdx.x / xcds, q = tiles / xcds, r = tiles % xcds;
    const uint32_t t = x * q + (x < r ? x : r) + wi;
    const uint32_t per_group = (uint32_t)p.group_m * tiles_n;      // (<= tiles)
    const uint32_t grp = t / per_group, rr = t % per_group, first = grp * (uint32_t)p.group_m;
    const uint32_t gm = tiles_m - first < (uint32_t)p.group_m ? tiles_m - first : (uint32_t)p.group_m;
    tile_m = first + rr % gm;
    tile_n = rr / gm;
}

// Fills in the tile counts and the raster.
void gemm_f32_raster(GemmF32Params& p, int64_t tiles_m, int64_t tiles_n, int BM, int BN, const DeviceInfo& dev);
// The sum of the k-splits in index order, then the epilogue.
hipError_t launch_splitk_reduce(const GemmF32Params& p, int epilogue, hipStream_t stream);

// The kernel on three bf16 terms where it takes the contraction (otherwise the duration is beyond all others); the combination
// of operand layouts and epilogue must be one of launch_gemm_f32.
GemmF32Plan gemm_f32x3_plan(const GemmF32Args& a, int max_split);
double gemm_f32x3_least_us();      // that it estimates for any contraction
hipError_t launch_gemm_f32x3(const GemmF32Args& a, GemmF32Params p, const GemmF32Plan& plan, hipStream_t stream);

}  // namespace sfb
