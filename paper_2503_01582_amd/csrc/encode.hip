// Multi-resolution hash encoding, forward (Sec. III-B "Object-level NeRFs":
// sample positions are normalised and encoded with the hash grid of Mueller
// et al. 2022 before the MLP).  The backward lives in scatter.hip.
//
// Layout: tables [L][T][2] (one float2 per row), features y level-major
// [L][n_samples][2], so a wavefront of one level writes 64 consecutive float2
// (512 contiguous bytes).  One thread per (sample, level): 8 corner rows,
// gathered from memory (grid: sample blocks, levels) or, where a level's table
// fits, from LDS.
#include <type_traits>

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

// Encoding from LDS: a block stages a level's rows and encodes a long run of
// samples against them.  The gathers above are bound by the lines the L1 caches
// fetch, about 600 cycles of a CU for 64 samples of a level; from LDS the same
// corners cost 125, the vector instructions that find and weigh them.  A table of
// up to 256 KB takes two passes, one feature of its rows at a time: twice the
// arithmetic (and half-line stores), still below the gathers.  The same products
// in the same order, so the same bits.  Measured on gfx950 (us), gathers against
// staged: 64777 rays x 33, FP32, 8 levels of 2^14 rows 125 / 54, 12 levels of
// 2^15 (two passes) 248 / 185; FP16, 12 levels of 2^15 243 / 84, 16 of 2^16 (two
// passes) 393 / 226; 48 objects with FP16 tables 11440 / 7863.  A run has to pay
// for staging its level, 3 us a pass and 128 KB: 2048 rays x 33, 8 levels of 2^14
// (2112 samples a CU) 12.4 / 10.0, 512 rays 7.0 / 7.4; in two passes 12288 rays x
// 33, 12 levels of 2^15 55 / 50, 4096 rays 23 / 31.  Longer runs than kLdsMost
// leave the last round of blocks emptier (256000 rays: 191 against 239 with
// 131072).
constexpr int kLdsThreads = 1024;
constexpr uint32_t kLdsBytes = 128 * 1024;
constexpr int64_t kLdsMost = 49152;                     // samples per staged level
constexpr int64_t kLdsMinRun = 1024, kLdsMinRun2 = 16384;  // fewest that pay for it, in one pass and two

// Passes over the samples that a level of 2^log2T rows needs: 1 if its rows fit
// the staged bytes, 2 if one feature of each does, else 0 (not staged).
__host__ __device__ constexpr int lds_planes(uint32_t row_bytes, int log2T)
{
    const uint64_t bytes = (uint64_t)row_bytes << log2T;
    return bytes < 64 ? 0 : bytes <= kLdsBytes ? 1 : bytes <= 2 * kLdsBytes ? 2 : 0;
}

template <typename Row>
struct Feature;
template <>
struct Feature<float2> {
    typedef float type;
    typedef float2 out;  // one feature of the rows in 16 bytes
    __device__ static float2 pick(uint4 v, int f)
    {
        return f ? make_float2(__uint_as_float(v.y), __uint_as_float(v.w))
                 : make_float2(__uint_as_float(v.x), __uint_as_float(v.z));
    }
};
template <>
struct Feature<half2_t> {
    typedef _Float16 type;
    typedef uint2 out;
    __device__ static uint2 pick(uint4 v, int f)
    {
        return f ? make_uint2((v.x >> 16) | (v.y & 0xffff0000u), (v.z >> 16) | (v.w & 0xffff0000u))
                 : make_uint2((v.x & 0xffffu) | (v.y << 16), (v.z & 0xffffu) | (v.w << 16));
    }
};

// Samples [s0, s1) of one level; gs0: the global index of sample s0.
template <typename Row, int kPlanes>
__device__ __forceinline__ void encode_lds(uint4* __restrict__ smem, const GridInfo& g, int l,
                                           const Row* __restrict__ level_table, const float* __restrict__ ray_obj,
                                           const float* __restrict__ t, int64_t gs0, uint32_t n, int32_t S,
                                           float inv_S, float2* __restrict__ y)
{
    const uint32_t side = (uint32_t)g.res[l] + 1u;
    const uint32_t rows = (g.dense_mask >> l) & 1u ? side * side * side : 1u << g.log2_table;
    const uint32_t vecs = (rows * (uint32_t)sizeof(Row) + 15u) / 16u;  // (a level's slice holds whole vectors)
    const uint4* src = reinterpret_cast<const uint4*>(level_table);
    const uint32_t ray0 = (uint32_t)gs0 / (uint32_t)S, off = (uint32_t)gs0 - ray0 * (uint32_t)S;
    const float* ro0 = ray_obj + 6 * (int64_t)ray0;
    t += gs0;
    auto corners = [&](uint32_t i, Corners& c) {
        const float* ro = ro0 + 6u * (uint32_t)(((float)(off + i) + 0.5f) * inv_S);
        const float ts = t[i];
        level_corners<true>(g, l, sample_coord(ts, ro[3], ro[0]), sample_coord(ts, ro[4], ro[1]),
                            sample_coord(ts, ro[5], ro[2]), c);
    };
    if constexpr (kPlanes == 1) {
#pragma unroll 8
        for (uint32_t i = threadIdx.x; i < vecs; i += kLdsThreads) smem[i] = src[i];
        __syncthreads();
        const Row* tab = reinterpret_cast<const Row*>(smem);
#pragma unroll 2
        for (uint32_t i = threadIdx.x; i < n; i += kLdsThreads) {
            Corners c;
            corners(i, c);
            y[i] = gather_blend_rows(tab, c);
        }
    } else {
        typedef Feature<Row> F;
        typename F::out* dst = reinterpret_cast<typename F::out*>(smem);
        const typename F::type* tab = reinterpret_cast<const typename F::type*>(smem);
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            if (f) __syncthreads();
#pragma unroll 8
            for (uint32_t i = threadIdx.x; i < vecs; i += kLdsThreads) dst[i] = F::pick(src[i], f);
            __syncthreads();
#pragma unroll 2
            for (uint32_t i = threadIdx.x; i < n; i += kLdsThreads) {
                Corners c;
                corners(i, c);
                float v[8], acc = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (float)tab[c.row[e]];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = fmaf(c.w[e], v[e], acc);
                reinterpret_cast<float*>(y)[2 * i + f] = acc;
            }
        }
    }
}

template <typename Row, int kPlanes>
__global__ __launch_bounds__(kLdsThreads) void k_encode_samples_lds(GridInfo g, const Row* __restrict__ table,
                                                                  const float* __restrict__ ray_obj,
                                                                  const float* __restrict__ t, int64_t n_s,
                                                                  int64_t run, int32_t S, float inv_S,
                                                                  float2* __restrict__ y)
{
    extern __shared__ uint4 smem[];
    const int l = blockIdx.y;
    const int64_t s0 = (int64_t)blockIdx.x * run;
    const uint32_t n = (uint32_t)(n_s - s0 < run ? n_s - s0 : run);
    encode_lds<Row, kPlanes>(smem, g, l, table + ((int64_t)l << g.log2_table), ray_obj, t, s0, n, S, inv_S,
                             y + (int64_t)l * n_s + s0);
}

// Object of an item of a batched launch: the last whose first item (`off` of its
// geometry) is not past it; objects without items have their successor's.
__device__ __forceinline__ int item_object(const ScatterObj* __restrict__ sobjs, int n_obj,
                                           int64_t ScatterObj::*off, int64_t item)
{
    int lo = 0, hi = n_obj - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sobjs[mid].*off <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Batched, staged objects: one block per item (object, level, run of samples).
__global__ __launch_bounds__(kLdsThreads) void k_encode_batch_lds(const ObjDev* __restrict__ objs,
                                                                const ScatterObj* __restrict__ sobjs, int n_obj,
                                                                const float* __restrict__ params,
                                                                const half2_t* __restrict__ params_f16,
                                                                const float* __restrict__ ray_obj,
                                                                const float* __restrict__ t, int32_t S, float inv_S,
                                                                float2* __restrict__ y)
{
    extern __shared__ uint4 smem[];
    const int64_t item = blockIdx.x;
    const int k = item_object(sobjs, n_obj, &ScatterObj::lds_off, item);
    const ScatterObj& so = sobjs[k];
    const ObjDev& o = objs[k];
    const uint32_t rem = (uint32_t)(item - so.lds_off);
    const int l = (int)(rem / (uint32_t)so.n_runs);
    const int64_t s0 = (int64_t)(rem - (uint32_t)l * (uint32_t)so.n_runs) * so.run;
    const uint32_t n = (uint32_t)(so.n_s - s0 < so.run ? so.n_s - s0 : so.run);
    const int64_t row0 = (int64_t)l << o.grid.log2_table, gs0 = so.s_begin + s0;
    float2* out = y + o.y_off / 2 + (int64_t)l * so.n_s + s0;
    auto encode = [&](auto* table) {
        typedef std::remove_const_t<std::remove_pointer_t<decltype(table)>> Row;
        if (lds_planes(sizeof(Row), o.grid.log2_table) == 1)
            encode_lds<Row, 1>(smem, o.grid, l, table, ray_obj, t, gs0, n, S, inv_S, out);
        else
            encode_lds<Row, 2>(smem, o.grid, l, table, ray_obj, t, gs0, n, S, inv_S, out);
    };
    if (o.table_dtype == PRENOM_F16)
        encode(params_f16 + o.param_off / 2 + row0);
    else
        encode(reinterpret_cast<const float2*>(params + o.param_off) + row0);
}

// Batched, the other objects: one block per item (object, level, block of
// kScatterBlockSamples samples); sobjs[i] and objs[i] describe object i.
__global__ __launch_bounds__(kScatterBlockSamples) void k_encode_batch(const ObjDev* __restrict__ objs,
                                                                   const ScatterObj* __restrict__ sobjs, int n_obj,
                                                                   const float* __restrict__ params,
                                                                   const half2_t* __restrict__ params_f16,
                                                                   const float* __restrict__ ray_obj,
                                                                   const float* __restrict__ t, int32_t S,
                                                                   uint32_t n_items, int run_log2,
                                                                   float2* __restrict__ y)
{
    const int64_t item = xcd_item(blockIdx.x, run_log2);
    if (item >= n_items) return;
    const int lo = item_object(sobjs, n_obj, &ScatterObj::item_off, item);
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
// position: the correctly rounded FP32 quotient is the same number, as rounding a
// quotient of two FP32 numbers to FP64 first changes nothing.  Used to refresh the
// density prior from the NeRF.  An XCD (blocks go to the 8 in turn) takes whole
// levels, a coarse one with a fine one, so that its L2 fetches an eighth of the
// tables instead of all of them; 64^3 vertices, 16 levels of 2^19 rows 71 -> 66 us,
// and 74 with FP64 quotients and 64-bit divisions.
template <typename Row>
__global__ __launch_bounds__(kEncBlock) void k_encode_grid(GridInfo g, const Row* __restrict__ table, uint32_t R,
                                                           int64_t p0, int64_t cnt, float2* __restrict__ y)
{
    const uint32_t n_blocks = (uint32_t)((cnt + kEncBlock - 1) / kEncBlock);
    const uint32_t item = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int turn = (int)(item / n_blocks);  // levels in the order 0, L - 1, 1, L - 2, ...
    if (turn >= g.n_levels) return;
    const int l = turn & 1 ? g.n_levels - 1 - (turn >> 1) : turn >> 1;
    const int64_t q = (int64_t)(item - (uint32_t)turn * n_blocks) * kEncBlock + threadIdx.x;
    if (q >= cnt) return;
    const uint32_t p = (uint32_t)(p0 + q), row = p / R, k = row / R;  // (R^3 <= 2^27)
    const float d = (float)(R - 1u);
    Corners c;
    level_corners(g, l, (float)(p - row * R) / d, (float)(row - k * R) / d, (float)k / d, c);
    const Row* lt = table + ((int64_t)l << g.log2_table);
    y[(int64_t)l * cnt + q] = gather_blend<true>(lt, g, l, c);
}

// out[p] = sigma of head output p (sc rows are (sigma, r, g, b)).
__global__ __launch_bounds__(256) void k_density_grid(const float4* __restrict__ sc, int64_t n, float* __restrict__ out)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p < n) out[p] = sc[p].x;
}

template <typename Row, int kPlanes>
hipError_t encode_samples_lds(const GridInfo& g, const Row* table, const float* ray_obj, const float* t, int64_t n_s,
                              int64_t run, int32_t S, float2* y, hipStream_t s)
{
    auto kern = k_encode_samples_lds<Row, kPlanes>;
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((uint32_t)((n_s + run - 1) / run), (uint32_t)g.n_levels), dim3(kLdsThreads),
                       kLdsBytes, s, g, table, ray_obj, t, n_s, run, S, 1.0f / (float)S, y);
    return hipGetLastError();
}

int64_t round_up(int64_t n, int64_t m) { return (n + m - 1) / m * m; }

dim3 enc_grid(int64_t n, int L) { return dim3((uint32_t)((n + kEncBlock - 1) / kEncBlock), (uint32_t)L); }

// Samples per staged block for `work` (level, sample) pairs: whole rounds of one
// block a CU, at most kLdsMost each.
int64_t lds_run(int64_t work)
{
    if (work == 0) return 0;
    const int64_t rounds = (work + kCus * kLdsMost - 1) / (kCus * kLdsMost);
    return (work + kCus * rounds - 1) / (kCus * rounds);
}

// Whether blocks of `run` samples pay for their staging.
bool lds_pays(int planes, int64_t run) { return planes && run >= (planes == 1 ? kLdsMinRun : kLdsMinRun2); }

template <typename Row>
hipError_t encode_samples(const GridInfo& g, const Row* table, const float* ray_obj, const float* t, int64_t n_s,
                          int32_t S, float2* y, hipStream_t s)
{
    const int planes = ((uintptr_t)table & 15) == 0 ? lds_planes(sizeof(Row), g.log2_table) : 0;
    if (lds_pays(planes, lds_run(n_s * g.n_levels))) {
        const int64_t rounds = (n_s * g.n_levels + kCus * kLdsMost - 1) / (kCus * kLdsMost);
        const int64_t per_level = rounds * kCus / g.n_levels;  // blocks (L <= 16)
        const int64_t run = round_up((n_s + per_level - 1) / per_level, 64);
        return planes == 1 ? encode_samples_lds<Row, 1>(g, table, ray_obj, t, n_s, run, S, y, s)
                           : encode_samples_lds<Row, 2>(g, table, ray_obj, t, n_s, run, S, y, s);
    }
    hipLaunchKernelGGL(k_encode_samples<Row>, enc_grid(n_s, g.n_levels), dim3(kEncBlock), 0, s, g, table, ray_obj, t,
                       n_s, S, y);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_encode_samples(const GridInfo& g, const float* table, const void* table_f16,
                                 const float* ray_obj, const float* t, int64_t n_rays, int32_t S, float* y,
                                 hipStream_t s)
{
    const int64_t n_s = n_rays * S;
    if (n_s == 0) return hipSuccess;
    return table_f16 ? encode_samples(g, (const half2_t*)table_f16, ray_obj, t, n_s, S, (float2*)y, s)
                     : encode_samples(g, (const float2*)table, ray_obj, t, n_s, S, (float2*)y, s);
}

hipError_t launch_encode_grid(const GridInfo& g, const float* table, const void* table_f16, int32_t R, int64_t p0,
                              int64_t cnt, float* y, hipStream_t s)
{
    if (cnt == 0) return hipSuccess;
    const dim3 grid((uint32_t)round_up((cnt + kEncBlock - 1) / kEncBlock * g.n_levels, 8));
    if (table_f16)
        hipLaunchKernelGGL(k_encode_grid<half2_t>, grid, dim3(kEncBlock), 0, s, g,
                           (const half2_t*)table_f16, (uint32_t)R, p0, cnt, (float2*)y);
    else
        hipLaunchKernelGGL(k_encode_grid<float2>, grid, dim3(kEncBlock), 0, s, g,
                           (const float2*)table, (uint32_t)R, p0, cnt, (float2*)y);
    return hipGetLastError();
}

hipError_t launch_density_grid(const float* sc, int64_t n, float* out, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_density_grid, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, (const float4*)sc, n, out);
    return hipGetLastError();
}

// With runs of a fixed length a launch of fewer items than 8 of them leaves XCDs
// without work; runs of at most a 32nd of the items give none of them more than a
// quarter above its share, and 256 items are as long as helps.  Measured on gfx950
// (us; runs of one, of an 8th, a 32nd and a 64th of the items, of 256): 512 items,
// 2^17 rows 14.4 / 10.1 / 11.3 / 13.1 / 24.0, 2^14 rows 9.0 / 9.2 / 9.2 / 9.0 / 19.7;
// 2304 items 47.0 / 42.4 / 35.0 / 32.6 / 42.5; 3760 76.6 / 48.7 / 49.4 / 52.2 / 48.7;
// 8192 126.5 / 108.1 / 107.8 / 101.9 / 107.8; 16384 and more within 2%.
int xcd_run_log2(int64_t n_items)
{
    int r = 0;
    while (r < 8 && ((int64_t)64 << r) <= n_items) ++r;
    return r;
}

void encode_split(const ObjDev* objs, ScatterObj* sobjs, int n_obj, int64_t& n_items, int64_t& n_lds)
{
    auto planes = [&](int i) {
        return lds_planes(objs[i].table_dtype == PRENOM_F16 ? 4 : 8, objs[i].grid.log2_table);
    };
    // The run of all objects that could be staged; if it is too short for those of
    // two passes, that of the others.
    auto run_of = [&](int most) {
        int64_t work = 0;
        for (int i = 0; i < n_obj; ++i)
            if (planes(i) && planes(i) <= most) work += sobjs[i].n_s * sobjs[i].grid.n_levels;
        return lds_run(work);
    };
    const int most = lds_pays(2, run_of(2)) ? 2 : 1;
    const int64_t run = run_of(most);
    n_items = n_lds = 0;
    for (int i = 0; i < n_obj; ++i) {
        ScatterObj& o = sobjs[i];
        o.item_off = n_items;
        o.lds_off = n_lds;
        o.n_runs = 0;
        o.run = 0;
        if (o.n_s > 0 && planes(i) <= most && lds_pays(planes(i), run)) {
            const int64_t runs = (o.n_s + run - 1) / run;  // even ones
            o.run = round_up((o.n_s + runs - 1) / runs, 64);
            o.n_runs = (int32_t)((o.n_s + o.run - 1) / o.run);
            n_lds += (int64_t)o.n_runs * o.grid.n_levels;
        } else {
            n_items += scatter_items(o);
        }
    }
}

hipError_t launch_encode_batch(const ObjDev* objs, const ScatterObj* sobjs, int n_obj, int64_t n_items, int64_t n_lds,
                               const float* params, const void* params_f16, const float* ray_obj, const float* t,
                               int32_t S, float* y, hipStream_t s)
{
    if (n_lds > 0) {
        hipError_t e = hipFuncSetAttribute((const void*)k_encode_batch_lds, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           kLdsBytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_encode_batch_lds, dim3((uint32_t)n_lds), dim3(kLdsThreads), kLdsBytes, s, objs, sobjs,
                           n_obj, params, (const half2_t*)params_f16, ray_obj, t, S, 1.0f / (float)S, (float2*)y);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (n_items == 0) return hipSuccess;
    const int run_log2 = xcd_run_log2(n_items);
    const dim3 grid((uint32_t)round_up(n_items, (int64_t)kXcds << run_log2));
    hipLaunchKernelGGL(k_encode_batch, grid, dim3(kScatterBlockSamples), 0, s, objs, sobjs, n_obj, params,
                       (const half2_t*)params_f16, ray_obj, t, S, (uint32_t)n_items, run_log2, (float2*)y);
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
