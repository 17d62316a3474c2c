// Multi-resolution hash encoding, forward (Sec. III-B "Object-level NeRFs":
// sample positions are normalised and encoded with the hash grid of Mueller
// et al. 2022 before the MLP).  The backward lives in scatter.hip.
//
// Layout: tables [L][T][2] (one float2 per row), features y level-major
// [L][n_samples][2], so a wavefront of one level writes 64 consecutive float2
// (512 contiguous bytes).  The launch grid is (sample blocks, levels): one
// thread per (sample, level), 8 float2 gathers each.
#include "common.h"

namespace prenom {
namespace {

constexpr int kEncBlock = 256;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float2 to_f2(float2 v) { return v; }
__device__ __forceinline__ float2 to_f2(half2_t v) { return make_float2((float)v[0], (float)v[1]); }

// Two consecutive table rows (an aligned row pair), and one row read through
// a buffer resource.
template <typename Row>
struct RowPair;
template <>
struct RowPair<float2> {
    typedef float4 type;
    struct __attribute__((packed, aligned(8))) any {  // two rows at any row's address
        float x, y, z, w;
    };
    __device__ static float2 lo(float4 v) { return make_float2(v.x, v.y); }
    __device__ static float2 hi(float4 v) { return make_float2(v.z, v.w); }
    __device__ static float2 lo(const any& v) { return make_float2(v.x, v.y); }
    __device__ static float2 hi(const any& v) { return make_float2(v.z, v.w); }
    __device__ static float2 row(__amdgpu_buffer_rsrc_t r, uint32_t off)
    {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
        return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
    }
};
template <>
struct RowPair<half2_t> {
    typedef half4_t type;
    struct __attribute__((packed, aligned(4))) any {
        half2_t a, b;
    };
    __device__ static float2 lo(const any& v) { return to_f2(v.a); }
    __device__ static float2 hi(const any& v) { return to_f2(v.b); }
    __device__ static float2 lo(half4_t v) { return make_float2((float)v[0], (float)v[1]); }
    __device__ static float2 hi(half4_t v) { return make_float2((float)v[2], (float)v[3]); }
    __device__ static float2 row(__amdgpu_buffer_rsrc_t r, uint32_t off)
    {
        const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
        return to_f2(__builtin_bit_cast(half2_t, v));
    }
};

// Raw buffer descriptor over `bytes` bytes at p (third word for the gfx9
// family: raw, untyped 32-bit data).  Loads at offsets past `bytes` return
// zero without a memory access.  p and bytes are the same in every lane (one
// level table per block); reading them from the first lane keeps the
// descriptor in scalar registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void* p, uint32_t bytes)
{
    // readfirstlane returns int: each word goes through uint32_t so that the
    // low word is zero-extended, not sign-extended, into the 64-bit address.
    const uint64_t a = (uint64_t)(uintptr_t)p;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint64_t u = ((uint64_t)hi << 32) | (uint64_t)lo;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uintptr_t)u), (short)0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}
constexpr uint32_t kOutOfRange = 0x80000000u;  // past any level table (T <= 2^24 rows of <= 8 bytes)

// Table rows are float2 (FP32 tables) or two halves (the FP16 copy).
// Plain gather: the 8 corner rows, all loads issued before the blend.
template <typename Row>
__device__ __forceinline__ float2 gather_blend_rows(const Row* __restrict__ level_table, const Corners& c)
{
    Row v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = level_table[c.row[e]];
    float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float2 f = to_f2(v[e]);
        acc.x = fmaf(c.w[e], f.x, acc.x);
        acc.y = fmaf(c.w[e], f.y, acc.y);
    }
    return acc;
}

// Paired gather.  Corners 2p and 2p + 1 differ only in x; on a hashed level
// their rows share an aligned row pair whenever x is even (x and x + 1 then
// hash to rows differing in bit 0 only).  Each pair is fetched as one aligned
// two-row load, plus a one-row buffer load whose offset is out of range (no
// memory access) in the lanes whose second corner lies inside that pair:
// about 1.5 cache-line requests per corner pair instead of 2, with no
// branches.  The blend adds the corners in the order e = 0..7 as above.
template <typename Row>
__device__ __forceinline__ float2 gather_blend_pairs(const Row* __restrict__ level_table, uint32_t n_rows,
                                                     const Corners& c)
{
    typedef RowPair<Row> RP;
    const __amdgpu_buffer_rsrc_t rsrc = raw_buffer(level_table, n_rows * (uint32_t)sizeof(Row));
    typename RP::type pv[4];
    float2 other[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {  // issue all loads first
        const uint32_t r0 = c.row[2 * p], r1 = c.row[2 * p + 1];
        pv[p] = *reinterpret_cast<const typename RP::type*>(level_table + (r0 & ~1u));
        other[p] = RP::row(rsrc, (r0 >> 1) != (r1 >> 1) ? r1 * (uint32_t)sizeof(Row) : kOutOfRange);
    }
    float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t r0 = c.row[2 * p], r1 = c.row[2 * p + 1];
        const float2 lo = RP::lo(pv[p]), hi = RP::hi(pv[p]);
        const float2 f0 = (r0 & 1u) ? hi : lo;
        const float2 f1 = (r0 >> 1) != (r1 >> 1) ? other[p] : ((r1 & 1u) ? hi : lo);
        acc.x = fmaf(c.w[2 * p], f0.x, acc.x);
        acc.y = fmaf(c.w[2 * p], f0.y, acc.y);
        acc.x = fmaf(c.w[2 * p + 1], f1.x, acc.x);
        acc.y = fmaf(c.w[2 * p + 1], f1.y, acc.y);
    }
    return acc;
}

// Dense levels: the rows of corners 2p and 2p + 1 follow each other, so each
// pair is one two-row load at the first row's address.
template <typename Row>
__device__ __forceinline__ float2 gather_blend_dense(const Row* __restrict__ level_table, const Corners& c)
{
    typedef RowPair<Row> RP;
    typename RP::any v[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) v[p] = *reinterpret_cast<const typename RP::any*>(level_table + c.row[2 * p]);
    // (keeps the compiler from joining these loads with the plain gather's,
    // which split them into their rows again)
    asm volatile("" ::: "memory");
    float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const float2 f0 = RP::lo(v[p]), f1 = RP::hi(v[p]);
        acc.x = fmaf(c.w[2 * p], f0.x, acc.x);
        acc.y = fmaf(c.w[2 * p], f0.y, acc.y);
        acc.x = fmaf(c.w[2 * p + 1], f1.x, acc.x);
        acc.y = fmaf(c.w[2 * p + 1], f1.y, acc.y);
    }
    return acc;
}

// The encoding is bound by the lines the L1 caches fetch: a wave's gather from
// 64 lines takes 150 cycles whether 4, 8 or 16 bytes are read from each (64
// bytes a cycle and CU), a gather that hits 40.  Hashed levels fetch four lines
// a sample however they are read (x and x + 1 lie in one line 15 times out of
// 16); reading them in pairs saves the hits.  Tables of fewer than
// 2^kPairMinLog2 rows hit more, and the pairs' selects cost more than they save.
// Measured on gfx950 (us): 65536 rays x 64 samples, 16 levels of 2^19 rows, 1167
// in pairs against 1297 plain; FP16 tables of 2^18 rows 1976 against 2058; 30011
// rays, 12 levels of 2^17, 317 against 306; a view over 2^15 rows 278 against
// 259.  The batch (kPairs false) reads hashed levels plainly, as one kernel
// serves tables of all sizes and types and the pairs' code costs the others: 24
// objects 3090 in pairs from 2^19 rows on against 2747 plain, 48 objects with
// FP16 tables 11344 against 11460.  Dense levels in pairs: 48 objects 11.9 ->
// 11.4 ms.
constexpr int kPairMinLog2 = 18;

template <bool kPairs, typename Row>
__device__ __forceinline__ float2 gather_blend(const Row* __restrict__ level_table, const GridInfo& g, int l,
                                               const Corners& c)
{
    if ((g.dense_mask >> l) & 1u) return gather_blend_dense(level_table, c);
    if (kPairs && g.log2_table >= kPairMinLog2) return gather_blend_pairs(level_table, 1u << g.log2_table, c);
    return gather_blend_rows(level_table, c);
}

template <typename Row>
__global__ __launch_bounds__(kEncBlock) void k_encode_samples(GridInfo g, const Row* __restrict__ table,
                                                              const float* __restrict__ ray_obj,
                                                              const float* __restrict__ t, int64_t n_s,
                                                              int32_t S, float2* __restrict__ y)
{
    const int64_t s = (int64_t)blockIdx.x * kEncBlock + threadIdx.x;
    const int l = blockIdx.y;
    if (s >= n_s) return;
    const float* ro = ray_obj + 6 * (int64_t)((uint32_t)s / (uint32_t)S);  // (n_s <= 2^29)
    const float ts = t[s];
    Corners c;
    level_corners(g, l, sample_coord(ts, ro[3], ro[0]), sample_coord(ts, ro[4], ro[1]),
                  sample_coord(ts, ro[5], ro[2]), c);
    const Row* lt = table + ((int64_t)l << g.log2_table);
    y[(int64_t)l * n_s + s] = gather_blend<true>(lt, g, l, c);
}

// Batched: one block per item (object, level, block of kScatterBlockSamples
// samples) of the batch's hash-table gradient (sobjs[i] and objs[i] describe
// object i).
__global__ __launch_bounds__(kScatterBlockSamples) void k_encode_batch(const ObjDev* __restrict__ objs,
                                                                   const ScatterObj* __restrict__ sobjs, int n_obj,
                                                                   const float* __restrict__ params,
                                                                   const half2_t* __restrict__ params_f16,
                                                                   const float* __restrict__ ray_obj,
                                                                   const float* __restrict__ t, int32_t S,
                                                                   float2* __restrict__ y)
{
    const int64_t item = blockIdx.x;
    int lo = 0, hi = n_obj - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sobjs[mid].item_off <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    const ScatterObj& so = sobjs[lo];
    const ObjDev& o = objs[lo];
    const uint32_t rem = (uint32_t)(item - so.item_off);
    const int l = (int)(rem / (uint32_t)so.n_blocks);
    const int bx = (int)(rem - (uint32_t)l * (uint32_t)so.n_blocks);
    const int64_t n_s = so.n_s;
    const int64_t s = (int64_t)bx * kScatterBlockSamples + threadIdx.x;
    if (s >= n_s) return;
    const int64_t gs = so.s_begin + s;
    const float* ro = ray_obj + 6 * (int64_t)((uint32_t)gs / (uint32_t)S);
    const float ts = t[gs];
    Corners c;
    level_corners(o.grid, l, sample_coord(ts, ro[3], ro[0]), sample_coord(ts, ro[4], ro[1]),
                  sample_coord(ts, ro[5], ro[2]), c);
    const int64_t row0 = (int64_t)l << o.grid.log2_table;  // rows of float2 / half2
    float2 v;
    if (o.table_dtype == PRENOM_F16)
        v = gather_blend<false>(params_f16 + o.param_off / 2 + row0, o.grid, l, c);
    else
        v = gather_blend<false>(reinterpret_cast<const float2*>(params + o.param_off) + row0, o.grid, l, c);
    y[o.y_off / 2 + (int64_t)l * n_s + s] = v;
}

__global__ __launch_bounds__(kEncBlock) void k_encode_points(GridInfo g, const float2* __restrict__ table,
                                                             const float* __restrict__ pos, int64_t n,
                                                             float2* __restrict__ y,
                                                             int32_t* __restrict__ corner_idx)
{
    const int64_t i = (int64_t)blockIdx.x * kEncBlock + threadIdx.x;
    const int l = blockIdx.y;
    if (i >= n) return;
    const float* p = pos + 3 * i;
    Corners c;
    level_corners(g, l, fminf(fmaxf(p[0], 0.0f), 1.0f), fminf(fmaxf(p[1], 0.0f), 1.0f),
                  fminf(fmaxf(p[2], 0.0f), 1.0f), c);
    const float2* lt = table + ((int64_t)l << g.log2_table);
    y[(int64_t)l * n + i] = gather_blend<true>(lt, g, l, c);
    if (corner_idx) {
        int32_t* ci = corner_idx + ((int64_t)l * n + i) * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) ci[e] = (int32_t)c.row[e];
    }
}

// Encoding of the R^3 grid vertices (i, j, k) / (R - 1), vertex p = (k R + j) R + i
// (x fastest); each coordinate is rounded from FP64 to FP32, like a sample
// position.  Used to refresh the density prior from the NeRF.
template <typename Row>
__global__ __launch_bounds__(kEncBlock) void k_encode_grid(GridInfo g, const Row* __restrict__ table, int32_t R,
                                                           int64_t p0, int64_t cnt, float2* __restrict__ y)
{
    const int64_t q = (int64_t)blockIdx.x * kEncBlock + threadIdx.x;
    const int l = blockIdx.y;
    if (q >= cnt) return;
    const int64_t p = p0 + q;
    const int64_t i = p % R, j = (p / R) % R, k = p / ((int64_t)R * R);
    const double d = (double)(R - 1);  // correctly rounded FP64 quotients, then FP32
    Corners c;
    level_corners(g, l, (float)((double)i / d), (float)((double)j / d), (float)((double)k / d), c);
    const Row* lt = table + ((int64_t)l << g.log2_table);
    y[(int64_t)l * cnt + q] = gather_blend<true>(lt, g, l, c);
}

// out[p] = sigma of head output p (sc rows are (sigma, r, g, b)).
__global__ __launch_bounds__(256) void k_density_grid(const float4* __restrict__ sc, int64_t n, float* __restrict__ out)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p < n) out[p] = sc[p].x;
}

dim3 enc_grid(int64_t n, int L) { return dim3((uint32_t)((n + kEncBlock - 1) / kEncBlock), (uint32_t)L); }

}  // namespace

hipError_t launch_encode_samples(const GridInfo& g, const float* table, const void* table_f16,
                                 const float* ray_obj, const float* t, int64_t n_rays, int32_t S, float* y,
                                 hipStream_t s)
{
    const int64_t n_s = n_rays * S;
    if (n_s == 0) return hipSuccess;
    if (table_f16)
        hipLaunchKernelGGL(k_encode_samples<half2_t>, enc_grid(n_s, g.n_levels), dim3(kEncBlock), 0, s, g,
                           (const half2_t*)table_f16, ray_obj, t, n_s, S, (float2*)y);
    else
        hipLaunchKernelGGL(k_encode_samples<float2>, enc_grid(n_s, g.n_levels), dim3(kEncBlock), 0, s, g,
                           (const float2*)table, ray_obj, t, n_s, S, (float2*)y);
    return hipGetLastError();
}

hipError_t launch_encode_grid(const GridInfo& g, const float* table, const void* table_f16, int32_t R, int64_t p0,
                              int64_t cnt, float* y, hipStream_t s)
{
    if (cnt == 0) return hipSuccess;
    if (table_f16)
        hipLaunchKernelGGL(k_encode_grid<half2_t>, enc_grid(cnt, g.n_levels), dim3(kEncBlock), 0, s, g,
                           (const half2_t*)table_f16, R, p0, cnt, (float2*)y);
    else
        hipLaunchKernelGGL(k_encode_grid<float2>, enc_grid(cnt, g.n_levels), dim3(kEncBlock), 0, s, g,
                           (const float2*)table, R, p0, cnt, (float2*)y);
    return hipGetLastError();
}

hipError_t launch_density_grid(const float* sc, int64_t n, float* out, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_density_grid, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, (const float4*)sc, n, out);
    return hipGetLastError();
}

hipError_t launch_encode_batch(const ObjDev* objs, const ScatterObj* sobjs, int n_obj, int64_t n_items,
                               const float* params, const void* params_f16, const float* ray_obj, const float* t,
                               int32_t S, float* y, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    hipLaunchKernelGGL(k_encode_batch, dim3((uint32_t)n_items), dim3(kScatterBlockSamples), 0, s, objs, sobjs, n_obj,
                       params, (const half2_t*)params_f16, ray_obj, t, S, (float2*)y);
    return hipGetLastError();
}

hipError_t launch_encode_points(const GridInfo& g, const float* table, const float* pos, int64_t n,
                                float* features, int32_t* corner_idx, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_encode_points, enc_grid(n, g.n_levels), dim3(kEncBlock), 0, s, g,
                       (const float2*)table, pos, n, (float2*)features, corner_idx);
    return hipGetLastError();
}

}  // namespace prenom
