// Helpers shared by the MLP kernels (FP32 and reduced-precision forms).
#pragma once

#include "common.h"

namespace prenom {

__device__ __forceinline__ floatx4 relu4(floatx4 v)
{
    floatx4 r;
    r[0] = fmaxf(v[0], 0.0f);
    r[1] = fmaxf(v[1], 0.0f);
    r[2] = fmaxf(v[2], 0.0f);
    r[3] = fmaxf(v[3], 0.0f);
    return r;
}

__device__ __forceinline__ floatx4 mask_pos(floatx4 g, floatx4 h)
{
    floatx4 r;
    r[0] = h[0] > 0.0f ? g[0] : 0.0f;
    r[1] = h[1] > 0.0f ? g[1] : 0.0f;
    r[2] = h[2] > 0.0f ? g[2] : 0.0f;
    r[3] = h[3] > 0.0f ? g[3] : 0.0f;
    return r;
}

// Orders one wave's LDS writes before its later LDS reads (and reads before
// later overwrites): a wave's LDS operations execute in program order, so
// only compiler reordering has to be prevented.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

// Per-block LDS and launch parameters of the backward kernels.
constexpr int kBwdWaves = 8;      // waves per block
constexpr int kBwdMaxBlocks = 256;

// Blocks of the backward grid for n_s samples (each block writes one partial dW).
inline int bwd_blocks(int64_t n_s)
{
    const int64_t n_tiles = (n_s + 15) / 16;
    int64_t b = (n_tiles + kBwdWaves * 2 - 1) / (kBwdWaves * 2);  // two tiles per wave
    b = b < 1 ? 1 : b;
    return (int)(b > kBwdMaxBlocks ? kBwdMaxBlocks : b);
}

// Blocks of a forward grid (and of the FP32 128-wide chain) whose blocks stage
// `lds` bytes of weight fragments before their first tile.  A block's staging is
// paid once however many tiles it walks, so the grid is the number of blocks that
// share the chip at once, 256 CUs times one to four by their LDS, and the tiles are
// dealt out evenly; a small launch keeps one tile a wave, the most CUs.  With up to
// 2048 blocks instead, 4096 rays x 32 (128-wide, two layers): FP32 132 -> 84 us, BF16
// 87 -> 39; 64-wide: FP32 47 -> 35; 65536 rays x 32: 128-wide FP32 1029 -> 920, BF16
// 220 -> 199, 32-wide FP32 123 -> 114.  Fewer still leave SIMDs without waves: 64-wide
// FP32 at 65536 rays with 512 blocks 331, with 1024 300.
inline int64_t fwd_blocks(int64_t n_tiles, int waves, size_t lds)
{
    const size_t fit = (size_t)120 * 1024 / (lds ? lds : 1);
    const int64_t most = kCus * (int64_t)(fit < 1 ? 1 : fit > 4 ? 4 : fit);
    const int64_t per = (n_tiles + waves * most - 1) / (waves * most);
    return (n_tiles + waves * per - 1) / (waves * per);
}

// Stage the tile's delta (D layout, out tiles) and h (D layout) for the
// dW = delta h^T contraction over the 16 samples.
template <int OTILES, int ITILES, int DP, int HP>
__device__ __forceinline__ void stage_dw(float* __restrict__ sD, float* __restrict__ sH,
                                         const floatx4 (&delta)[OTILES], const floatx4 (&h)[ITILES], int q, int j)
{
#pragma unroll
    for (int to = 0; to < OTILES; ++to)
#pragma unroll
        for (int r = 0; r < 4; ++r) sD[j * DP + 16 * to + 4 * q + r] = delta[to][r];
#pragma unroll
    for (int ti = 0; ti < ITILES; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r) sH[j * HP + 16 * ti + 4 * q + r] = h[ti][r];
}

// Add (or, for the first wave, store) one dW accumulator set into the
// block's LDS reduction buffer (D layout: row 16 to + 4 q + r, col 16 ti + j).
template <int OTILES, int ITILES>
__device__ __forceinline__ void merge_dw(float* __restrict__ dst, const floatx4 (&dw)[OTILES][ITILES], int rows,
                                         int cols, int q, int j, bool first)
{
#pragma unroll
    for (int to = 0; to < OTILES; ++to)
#pragma unroll
        for (int ti = 0; ti < ITILES; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * to + 4 * q + r, col = 16 * ti + j;
                if (row < rows && col < cols) {
                    float* p = dst + row * cols + col;
                    *p = first ? dw[to][ti][r] : *p + dw[to][ti][r];
                }
            }
}

// ---------------------------------------------------------------- 128-wide weight gradient
// The weight-gradient kernel of the 128-wide FP32 MLP stages a chunk of
// kDwChunk samples in LDS: every layer's delta and activation rows (pitch PW
// floats), the input features (pitch PY, zero beyond IN) and the head adjoint
// dO, all loaded with coalesced vector reads; the MFMA operands are then read
// from LDS.  Lanes q step one sample, so PW = 16 mod 64 keeps those reads free of
// bank conflicts.
constexpr int kDwChunk = 32;

template <int W, int D, int PW, int PY>
struct DwStage {
    static constexpr int DL = 0;                          // deltas [D][chunk][PW]
    static constexpr int AC = DL + D * kDwChunk * PW;     // activations [D][chunk][PW]
    static constexpr int Y = AC + D * kDwChunk * PW;      // inputs [chunk][PY]
    static constexpr int DO = Y + kDwChunk * PY;          // head adjoint [chunk][4]
    static constexpr int FLOATS = DO + kDwChunk * 4;
};

// Staging of samples [s0, min(s0 + kDwChunk, s_end)) in two halves: dw_load
// reads a thread's share into registers, dw_store writes it to LDS (zeros past
// the end; input columns >= IN zero).  y: level-major [L][n_s][2]; act, dlt: rows
// of W floats, [D][n_s][W].  kDwThreads threads.
constexpr int kDwThreads = 256;

template <int W, int D, int PY>
struct DwRegs {
    static constexpr int V = W / 4;  // float4 per row
    static constexpr int N_ROW = D * kDwChunk * V, PER = N_ROW / kDwThreads;
    static constexpr int N_Y = kDwChunk * (PY / 2), PER_Y = N_Y / kDwThreads;
    static_assert(N_ROW % kDwThreads == 0 && N_Y % kDwThreads == 0, "whole shares");
    floatx4 a[PER], d[PER];
    float2 yv[PER_Y];
    float4 g, v;  // head adjoint inputs of one sample (threads < kDwChunk)
};

template <int IN, int W, int D, int PY>
__device__ __forceinline__ void dw_load(DwRegs<W, D, PY>& R, const float* __restrict__ y, const float4* __restrict__ sc,
                                        const float4* __restrict__ dout, const float* __restrict__ act,
                                        const float* __restrict__ dlt, int64_t n_s, int64_t s0, int64_t s_end)
{
    using Rg = DwRegs<W, D, PY>;
#pragma unroll
    for (int u = 0; u < Rg::PER; ++u) {
        const int i = threadIdx.x + kDwThreads * u;
        const int k = i / (kDwChunk * Rg::V), rem = i % (kDwChunk * Rg::V), r = rem / Rg::V, c = rem % Rg::V;
        const int64_t s = s0 + r;
        R.a[u] = R.d[u] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (s < s_end) {
            R.a[u] = *reinterpret_cast<const floatx4*>(act + ((int64_t)k * n_s + s) * W + 4 * c);
            R.d[u] = *reinterpret_cast<const floatx4*>(dlt + ((int64_t)k * n_s + s) * W + 4 * c);
        }
    }
#pragma unroll
    for (int u = 0; u < Rg::PER_Y; ++u) {
        const int i = threadIdx.x + kDwThreads * u, r = i / (PY / 2), l = i % (PY / 2);
        const int64_t s = s0 + r;
        R.yv[u] = s < s_end && 2 * l < IN ? reinterpret_cast<const float2*>(y)[(int64_t)l * n_s + s]
                                          : make_float2(0.0f, 0.0f);
    }
    const int64_t s = s0 + threadIdx.x;
    const bool ok = threadIdx.x < kDwChunk && s < s_end;
    R.g = ok ? dout[s] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    R.v = ok ? sc[s] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

template <int W, int D, int PW, int PY>
__device__ __forceinline__ void dw_store(float* __restrict__ lds, const DwRegs<W, D, PY>& R)
{
    using St = DwStage<W, D, PW, PY>;
    using Rg = DwRegs<W, D, PY>;
#pragma unroll
    for (int u = 0; u < Rg::PER; ++u) {
        const int i = threadIdx.x + kDwThreads * u;
        const int k = i / (kDwChunk * Rg::V), rem = i % (kDwChunk * Rg::V), r = rem / Rg::V, c = rem % Rg::V;
        *reinterpret_cast<floatx4*>(lds + St::AC + (k * kDwChunk + r) * PW + 4 * c) = R.a[u];
        *reinterpret_cast<floatx4*>(lds + St::DL + (k * kDwChunk + r) * PW + 4 * c) = R.d[u];
    }
#pragma unroll
    for (int u = 0; u < Rg::PER_Y; ++u) {
        const int i = threadIdx.x + kDwThreads * u, r = i / (PY / 2), l = i % (PY / 2);
        *reinterpret_cast<float2*>(lds + St::Y + r * PY + 2 * l) = R.yv[u];
    }
    if (threadIdx.x < kDwChunk) {  // d sigma / d o0 = sigma, d c / d o = c (1 - c)
        const float4 g = R.g, v = R.v;
        *reinterpret_cast<floatx4*>(lds + St::DO + threadIdx.x * 4) =
            floatx4{g.x * v.x, g.y * v.y * (1.0f - v.y), g.z * v.z * (1.0f - v.z), g.w * v.w * (1.0f - v.w)};
    }
}

}  // namespace prenom
