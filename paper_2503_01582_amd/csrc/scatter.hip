// Hash-table gradient without global atomics: a bucketed scatter-add.
//
// The backward of the encoding adds w_e * dy to the table row of each of the
// 8 cell corners of every (sample, level).  On gfx950 every global FP32
// atomic costs about the same whatever its scope (a device-wide ceiling near
// 2e10 per second), so at 10^9 contributions per step they cannot be issued
// one by one.  Instead the contributions are bucketed by table tile (2^13 rows,
// whose accumulators fill 128 KB of LDS):
//
//   place  : one workgroup per item (level, block of 512 samples) computes the
//            block's contributions, sorts them by tile in LDS and writes them
//            to the item's own range of the record array, all tiles one after
//            another, with the start of every tile's segment and the block's
//            largest |dy|.  Nothing has to be known about the other blocks, so
//            no counting pass and no scan over blocks precede it, and the
//            write is one linear copy out of LDS
//   reduce : one workgroup per (tile, range of blocks) gathers the tile's
//            segments of those blocks, 16 lanes per segment, and accumulates
//            them in LDS; a tile with one range is added to the gradient rows
//            (the workgroup owns them), the others write their 64-bit sums
//            and the scale of these
//   combine: the sums of a tile's ranges added, in their order, and applied
//
// The LDS accumulation is 64-bit fixed point (integer LDS atomics run several
// times faster than FP32 ones), at a scale 2^e of the workgroup's own.  A row
// gets at most 512 max|dy| from a block, as the trilinear weights of a sample
// sum to 1, and at most 8 max|dy| from a record; with e chosen so that the
// smaller of the two, summed over the blocks, times 2^e < 2^62 no sum can
// overflow, and with one record's value times 2^e < 2^50 as well, each
// contribution is rounded by at most 2^-(e+1), far below FP32 resolution of the
// tile's larger rows however few of the level's records it holds.  Integer sums
// do not depend on order and the ranges' are added in one order, so the gradient
// is bit-reproducible.
//
// A record keeps 21 significant bits of the larger of its two features (an
// FP32 value has 24): each feature is within 2^-21 of the larger one's
// magnitude; the sum over records is then exact up to the fixed-point
// rounding.
//
// Corner rows and weights are computed by the same function as the forward
// encoding.
//
// The same kernels serve one object (its geometry passed by value) and a
// batch of objects with different grids (geometry in a device table): tiles,
// sample blocks and (object, level) pairs of all objects are numbered
// consecutively, so every phase is one launch for the whole batch.
#include "common.h"

namespace prenom {
namespace {

constexpr int kPlaceThreads = kScatterBlockSamples;
constexpr int kSamplesPerBlock = kPlaceThreads;  // one sample per thread
constexpr int kRecordsPerBlock = kSamplesPerBlock * 8;
constexpr int kReduceThreads = 1024;
constexpr int kSegLanes = 16;                           // lanes that read one segment
constexpr int kSegGroups = kReduceThreads / kSegLanes;  // segments in flight per workgroup
// Records in flight per lane: a step covers 80 records of a segment, so the
// segments of a 2^19-row level (4096 / 64 = 64 records on average) take one.
constexpr int kSegStep = 5;
// Blocks whose segment bounds a workgroup holds: in LDS at a time, and in registers
// from the pass that finds the scale (each thread's, kReduceThreads apart).
constexpr int kHeads = 2048, kHeldHeads = 8;
constexpr int kCombineThreads = 256;
// Reduce items of a pass (scatter_split): about kReduceItems of even size, so
// that the CUs stay busy to the end whatever the tables' sizes, but none
// smaller than kReduceMinRecords records, below which clearing and writing out
// the 128 KB of accumulators costs more than the records.
constexpr int64_t kReduceItems = 768;
constexpr int64_t kReduceMinRecords = 1 << 15;

// ---------------------------------------------------------------- records
// A record holds the row within the tile (bits 0-12), an exponent offset r
// (EB bits) and the two's-complement mantissas qx, qy (MB bits each); its
// value is (qx, qy) * 2^(E - r - (MB - 1)), E being the record exponent of
// its item (level, sample block).  A record whose larger feature lies below
// 2^(E - r), r at its largest, has fewer significant bits.  Two formats:
//   full:    EB = 7, MB = 22, one 64-bit word (21 significant bits);
//   compact: EB = 5, MB = 15, 48 bits kept as a 32-bit word (bits 0-31) in
//            one array and a 16-bit word (bits 32-47) in another (14
//            significant bits), for FP16 tables.
constexpr int kRecExpBits = 7;
constexpr int kRecMantBits = 22;
constexpr int kRecExpBitsC = 5;
constexpr int kRecMantBitsC = 15;
static_assert(kTileBits + kRecExpBitsC + 2 * kRecMantBitsC == 48, "compact record fields fill 48 bits");
static_assert(kTileBits + kRecExpBits + 2 * kRecMantBits == 64, "record fields fill one word");

// Record exponent E of a block whose largest |dy| is bm: a record sums at most
// 8 contributions w dy with 0 <= w <= 1, so |record| <= 8 bm < 2^(E - 1).
__device__ __forceinline__ int block_rec_exp(float bm)
{
    int e = 0;
    frexpf(bm, &e);  // bm < 2^e
    return e + 4;
}

// A record is encoded by a product with 2^(MB - 1 - E + r), which has to be a
// normal number: r goes up to E + 100, and a block with E below kTinyExp has its
// values multiplied by 2^kTinyUp first (exact; E then is within -48 and 51).  So
// r reaches 52 at least, unless its field ends before or no FP32 value needs as
// much, and what it does not reach is below the fixed point's rounding.
constexpr int kTinyExp = -44, kTinyUp = 96;

// max(|x|, |y|) in one instruction (fmaxf would first quiet both operands).
__device__ __forceinline__ float max_abs(float x, float y)
{
    float m;
    asm("v_max_f32_e64 %0, |%1|, |%2|" : "=v"(m) : "v"(x), "v"(y));
    return m;
}

// min(max(v, 0), hi) for hi >= 0 in one instruction.
__device__ __forceinline__ int clamp0(int v, int hi)
{
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(v), "v"(hi));
    return r;
}

// Words of the record (lo: bits 0-31, hi: the rest).  The mantissas are
// rounded to nearest by adding 1.5 * 2^23 (the sum's unit in the last place is
// 1, its low bits the two's complement of the integer); the larger one can
// round up to 2^(MB-1), one past the field: it is held at 2^(MB-1) - 1 (an
// error of one unit in its last place).  r_max: the largest exponent offset; a
// smaller record keeps it and fewer bits.
template <int EB, int MB>
__device__ __forceinline__ void encode_record(float2 v, int E, int r_max, uint32_t row, uint32_t& lo, uint32_t& hi)
{
    int k = 0;
    frexpf(max_abs(v.x, v.y), &k);  // 2^(k-1) <= larger feature < 2^k
    const uint32_t r = (uint32_t)clamp0(E - k, r_max);  // (a zero record has k = 0)
    const float scale = __uint_as_float((r << 23) + ((uint32_t)(MB - 1 + 127 - E) << 23));  // 2^(MB - 1 - E + r)
    constexpr float kMagic = 12582912.0f, kMax = (float)((1u << (MB - 1)) - 1u);
    const uint32_t bx = __float_as_uint(__builtin_amdgcn_fmed3f(fmaf(v.x, scale, kMagic), kMagic - kMax, kMagic + kMax));
    const uint32_t by = __float_as_uint(__builtin_amdgcn_fmed3f(fmaf(v.y, scale, kMagic), kMagic - kMax, kMagic + kMax));
    constexpr int kX = kTileBits + EB;      // first bit of qx
    constexpr int kXl = 32 - kX;            // its bits in the low word
    constexpr uint32_t kXh = (1u << (MB - kXl)) - 1u;
    lo = (bx << kX) | (r << kTileBits) | row;
    hi = ((bx >> kXl) & kXh) | (by << (MB - kXl));
}

// Fields of a record's words: row key, exponent offset, mantissas.
template <int EB, int MB>
__device__ __forceinline__ void decode_record(uint32_t lo, uint32_t hi, uint32_t& key, int& r, int& qx, int& qy)
{
    const uint64_t w = (uint64_t)hi << 32 | lo;
    key = lo & (kTileRows - 1);
    r = (int)((lo >> kTileBits) & ((1u << EB) - 1u));
    qx = (int)((uint32_t)(w >> (kTileBits + EB)) << (32 - MB)) >> (32 - MB);
    qy = (int)((uint32_t)(w >> (kTileBits + EB + MB)) << (32 - MB)) >> (32 - MB);
}

// q * 2^sh rounded to an integer (halves upward), for |q| <= 2^21 and sh <= 37
// (8 max|dy| times the scale is below 2^50, and a block's E at most 4 above the
// exponent of the largest: sh <= 51 - (MB - 1)).
__device__ __forceinline__ long long scale_mantissa(int q, int sh)
{
    const int d = min(40 - sh, 63);
    return (((long long)q << 40) + (1ll << (d - 1))) >> d;
}

// ---------------------------------------------------------------- object lookup
// Index of the last object whose `field` is <= v (fields ascend with the index).
template <bool kMany, typename F>
__device__ __forceinline__ int last_le(const ScatterArgs& a, int64_t v, F field)
{
    if constexpr (!kMany) {
        return 0;
    } else {
        int lo = 0, hi = a.n_obj - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (field(a.objs[mid]) <= v)
                lo = mid;
            else
                hi = mid - 1;
        }
        return lo;
    }
}

template <bool kMany>
__device__ __forceinline__ const ScatterObj& sobj(const ScatterArgs& a, int i)
{
    if constexpr (kMany)
        return a.objs[i];
    else
        return a.one;
}

// Last level whose first entry in `base` is <= v.
__device__ __forceinline__ int level_of(const int32_t* base, int n_levels, int v)
{
    int l = 0;
    while (l + 1 < n_levels && base[l + 1] <= v) ++l;
    return l;
}

// Sum and maximum over a wave by DPP (row shifts, whose lanes before the row's
// start read 0; then each row's last lane into the next rows): the last lane ends
// with them.  For values that are not negative; every lane must call them.
__device__ __forceinline__ float row_sum(float v)
{
    v += dpp_f32<0x111>(v);
    v += dpp_f32<0x112>(v);
    v += dpp_f32<0x114>(v);
    return v + dpp_f32<0x118>(v);
}

__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, dpp_f32<0x111>(v));
    v = fmaxf(v, dpp_f32<0x112>(v));
    v = fmaxf(v, dpp_f32<0x114>(v));
    return fmaxf(v, dpp_f32<0x118>(v));
}

__device__ __forceinline__ float wave_sum(float v)
{
    v = row_sum(v);
    v += dpp_f32<0x142>(v);
    return v + dpp_f32<0x143>(v);
}

__device__ __forceinline__ float wave_max(float v)
{
    v = row_max(v);
    v = fmaxf(v, dpp_f32<0x142>(v));
    return fmaxf(v, dpp_f32<0x143>(v));
}

// First entry of item (level l, block bx) of object o in the segment starts:
// tiles[l] + 1 of them per item.
__device__ __forceinline__ int64_t seg_index(const ScatterObj& o, int l, int bx)
{
    return o.seg_off + (int64_t)o.n_blocks * (o.tile_base[l] + l) + (int64_t)bx * (o.tiles[l] + 1);
}

// Dynamic LDS of the place kernel for levels of at most nt tiles: staged
// records, histogram (then segment starts, and the total).
__host__ __device__ constexpr size_t place_lds_bytes(int nt, bool compact)
{
    return (size_t)kRecordsPerBlock * (compact ? 6 : 8) + (size_t)(nt + 1) * 4;
}

// Place is bound by its vector instructions (ranks, record encoding, corner
// arithmetic).  A block's 4096 records fill 32 KB of LDS (24 KB compact), so
// four workgroups of eight waves share a CU.
template <bool kMany, bool kCompact>
__global__ __launch_bounds__(kPlaceThreads) void k_scatter_place(ScatterArgs a)
{
    constexpr int EB = kCompact ? kRecExpBitsC : kRecExpBits, MB = kCompact ? kRecMantBitsC : kRecMantBits;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_max;
    // full records; or compact ones: low words, then high words
    const uint64_t* s_rec = reinterpret_cast<const uint64_t*>(smem);
    const uint32_t* s_lo = reinterpret_cast<const uint32_t*>(smem);
    const uint16_t* s_hi = reinterpret_cast<const uint16_t*>(s_lo + kRecordsPerBlock);
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem + kRecordsPerBlock * (kCompact ? 6 : 8));
    const int64_t item = blockIdx.x;
    const ScatterObj& o = sobj<kMany>(a, last_le<kMany>(a, item, [](const ScatterObj& v) { return v.item_off; }));
    const uint32_t rem = (uint32_t)(item - o.item_off);
    const int l = (int)(rem / (uint32_t)o.n_blocks);
    const int bx = (int)(rem - (uint32_t)l * (uint32_t)o.n_blocks);
    const int nt = o.tiles[l];
    // Samples of the block, its first ray and the position of its first sample
    // on that ray; a lane's ray follows from its distance, below 2^10, by a
    // product with 1 / S (exact: the quotients' fractions stay 1 / (2 S) away
    // from an integer).  The gradient, t and the ray are loaded together and
    // the corners computed whatever dy is, so the loads are not serialised
    // behind a test.
    const int64_t s0 = (int64_t)bx * kSamplesPerBlock;
    const uint32_t n_in = (uint32_t)min((int64_t)kSamplesPerBlock, o.n_s - s0);
    const uint32_t gs0 = (uint32_t)(o.s_begin + s0);  // < 2^29 samples
    const uint32_t ray0 = gs0 / (uint32_t)a.S;
    const bool in = threadIdx.x < n_in;
    const uint32_t sl = min(threadIdx.x, n_in - 1u);
    const uint32_t lray = (uint32_t)(((float)(gs0 - ray0 * (uint32_t)a.S + sl) + 0.5f) * a.inv_S);
    const float* ro = a.ray_obj + 6 * (int64_t)ray0 + 6u * lray;
    float2 d = (a.dy + o.dy_off + (int64_t)l * o.n_s + s0)[sl];
    const float ts = (a.t + gs0)[sl];
    for (int i = threadIdx.x; i < nt; i += kPlaceThreads) hist[i] = 0;
    if (threadIdx.x == 0) s_max = 0u;
    Corners c;
    level_corners<true>(o.grid, l, sample_coord(ts, ro[3], ro[0]), sample_coord(ts, ro[4], ro[1]),
                  sample_coord(ts, ro[5], ro[2]), c);
    if (!in) d = make_float2(0.0f, 0.0f);
    // A non-finite feature gradient marks the step for the loss scaler, which
    // then skips the update, and contributes nothing: it would take the other
    // samples' scale, and their run sums (products with 0) if it lies beside them.
    const bool fx = isfinite(d.x), fy = isfinite(d.y);
    if (a.nonfinite && !(fx && fy)) a.nonfinite[0] = 1;
    d = make_float2(fx ? d.x : 0.0f, fy ? d.y : 0.0f);
    const bool has = d.x != 0.0f || d.y != 0.0f;
    // (runs whose sum could overflow stay apart)
    const bool start = run_head(c, has), head = __ballot(max_abs(d.x, d.y) >= 0x1p124f) ? has : start;
    float2 val[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        val[e] = make_float2(c.w[e] * d.x, c.w[e] * d.y);
    if (__ballot(has && !head)) run_sum(val, head || !has);
    const float m = wave_max(max_abs(d.x, d.y));
    __syncthreads();
    if ((threadIdx.x & 63) == 63) atomicMax(&s_max, __float_as_uint(m));  // (m >= 0: ordered as its bits)
    // Rank of each record within its tile (LDS atomics), in units of kUnit; the
    // histogram counts in those units, so that a segment's start and a rank add
    // up to the record's LDS address (compact: to its high word's).
    constexpr uint32_t kUnit = kCompact ? 2 : 8;
    uint32_t rank[8], tile[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[e] = c.row[e] >> kTileBits;
    if (head) {
        if (nt <= kAggregateTiles) {
#pragma unroll
            for (int e = 0; e < 8; ++e) rank[e] = wave_aggregated_add(hist, tile[e], kUnit);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) rank[e] = atomicAdd(&hist[tile[e]], kUnit);
        }
    }
    __syncthreads();
    const float bm = __uint_as_float(s_max);
    int E = __builtin_amdgcn_readfirstlane(block_rec_exp(bm));
    if (E < kTinyExp) {
        E += kTinyUp;
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = make_float2(val[e].x * 0x1p96f, val[e].y * 0x1p96f);
    }
    const int r_max = min((1 << EB) - 1, E + 100);
    // segment starts: exclusive scan of the histogram in place (by one wave)
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        uint32_t carry = 0;
        for (int base = 0; base < nt; base += 64) {
            const int i = base + lane;
            uint32_t v = i < nt ? hist[i] : 0u, incl = v;
#pragma unroll
            for (int dd = 1; dd < 64; dd <<= 1) {
                const uint32_t up = __shfl_up(incl, dd);
                if (lane >= dd) incl += up;
            }
            if (i < nt) hist[i] = carry + incl - v;
            carry += __shfl(incl, 63);
        }
        if (lane == 0) {
            hist[nt] = carry;
            a.block_max[item] = bm;
        }
    }
    __syncthreads();
    // stage the encoded records sorted by tile
    if (head) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t p = hist[tile[e]] + rank[e];
            uint32_t lo, hi;
            encode_record<EB, MB>(val[e], E, r_max, c.row[e] & (kTileRows - 1), lo, hi);
            if constexpr (kCompact) {
                *reinterpret_cast<uint32_t*>(smem + 2 * p) = lo;
                *reinterpret_cast<uint16_t*>(smem + kRecordsPerBlock * 4 + p) = (uint16_t)hi;
            } else {
                *reinterpret_cast<uint64_t*>(smem + p) = (uint64_t)hi << 32 | lo;
            }
        }
    }
    uint16_t* seg = a.seg + seg_index(o, l, bx);
    for (int i = threadIdx.x; i <= nt; i += kPlaceThreads) seg[i] = (uint16_t)(hist[i] / kUnit);
    __syncthreads();
    // the block's records to its range of the record array, 16 bytes per lane
    const uint32_t total = hist[nt] / kUnit;
    if constexpr (kCompact) {
        uint32_t* glo = reinterpret_cast<uint32_t*>(a.recs) + item * kRecordsPerBlock;
        uint16_t* ghi = reinterpret_cast<uint16_t*>(reinterpret_cast<uint32_t*>(a.recs) + a.n_records) +
                        item * kRecordsPerBlock;
        for (uint32_t p = threadIdx.x * 4; p < total; p += kPlaceThreads * 4)
            *reinterpret_cast<uint4*>(glo + p) = *reinterpret_cast<const uint4*>(s_lo + p);
        for (uint32_t p = threadIdx.x * 8; p < total; p += kPlaceThreads * 8)
            *reinterpret_cast<uint4*>(ghi + p) = *reinterpret_cast<const uint4*>(s_hi + p);
    } else {
        uint64_t* g = a.recs + item * kRecordsPerBlock;
        for (uint32_t p = threadIdx.x * 2; p < total; p += kPlaceThreads * 2)
            *reinterpret_cast<uint4*>(g + p) = *reinterpret_cast<const uint4*>(s_rec + p);
    }
}

// Largest e with bound * 2^e < 2^62 (on any row's sum; rounding the bound itself
// takes a part of the factor 2 that is left to 2^63) and 8 m * 2^e < 2^50 (on any
// record).  A bound beyond FP32 is below 2^157: 2^20 blocks of 2^9 * 2^128.
__device__ __forceinline__ int fixed_point_exp(float bound, float m)
{
    if (!(bound > 0.0f)) return 0;
    int ex = 157, evx = 0;
    if (isfinite(bound)) frexpf(bound, &ex);  // bound < 2^ex
    frexpf(m, &evx);                          // m < 2^evx
    return min(62 - ex, 47 - evx);
}

// One workgroup per reduce item: blocks [b0, b1) of one tile.  Its segments
// are read 16 lanes each (128 contiguous bytes a load), the next step's records
// requested before the current one's are added.  Bound by the LDS atomics
// (two 64-bit adds per record).  The scale needs all the segments' bounds before
// the first record: they are read at once and kept (ranges of more than 8192
// blocks read the others twice; reading them in turn, and all beyond the first
// 2048 twice, took 26 us of the 865 of 65536 rays x 64, 16 levels of 2^19 rows).
template <bool kMany, bool kCompact>
__global__ __launch_bounds__(kReduceThreads) void k_scatter_reduce(ScatterArgs a)
{
    constexpr int EB = kCompact ? kRecExpBitsC : kRecExpBits, MB = kCompact ? kRecMantBitsC : kRecMantBits;
    __shared__ unsigned long long acc[2 * kTileRows];  // fixed point: feature 0 rows, then feature 1 rows
    __shared__ uint2 head[kHeads];  // segments of kHeads blocks: start and end, max |dy| of the block
    __shared__ float2 w_part[kReduceThreads / 64];  // bound and maximum of a wave
    const int64_t ritem = blockIdx.x;
    const ScatterObj& o = sobj<kMany>(a, last_le<kMany>(a, ritem, [](const ScatterObj& v) { return v.ritem_off; }));
    const int rl = (int)(ritem - o.ritem_off);
    const int l = level_of(o.ritem_base, o.grid.n_levels, rl);
    const int n_split = o.split[l];
    const int tt = (rl - o.ritem_base[l]) / n_split;
    const int part = (rl - o.ritem_base[l]) - tt * n_split;
    const int nb = o.n_blocks;
    const int per = (nb + n_split - 1) / n_split;
    const int b0 = min(part * per, nb), b1 = min(b0 + per, nb);
    const int64_t row0 = (int64_t)tt << kTileBits;
    const int n_rows = (int)min((int64_t)kTileRows, o.level_rows[l] - row0);
    for (int i = threadIdx.x; i < n_rows; i += kReduceThreads) {
        acc[i] = 0ull;
        acc[kTileRows + i] = 0ull;
    }
    const int ln = threadIdx.x & (kSegLanes - 1);
    const int nt1 = o.tiles[l] + 1;
    const uint16_t* seg = a.seg + seg_index(o, l, 0) + tt;
    const int64_t item0 = o.item_off + (int64_t)l * nb;
    auto segment = [&](int b) {
        const uint16_t* p = seg + (int64_t)b * nt1;
        return make_uint2((uint32_t)p[0] | (uint32_t)p[1] << 16, __float_as_uint(a.block_max[item0 + b]));
    };
    const int n_range = b1 - b0;
    uint2 held[kHeldHeads];
#pragma unroll
    for (int u = 0; u < kHeldHeads; ++u) {
        const int i = (int)threadIdx.x + u * kReduceThreads;
        held[u] = make_uint2(0u, 0u);
        if (u * kReduceThreads < n_range && i < n_range) held[u] = segment(b0 + i);
    }
    float bound = 0.0f;  // of the rows' sums, and
    float m = 0.0f;      // the largest |dy| of the blocks that reach the tile
    auto note = [&](uint2 h) {
        const uint32_t n = (h.x >> 16) - (h.x & 0xffffu);
        const float bm = n ? __uint_as_float(h.y) : 0.0f;
        bound = fmaf((float)min(8u * n, (uint32_t)kSamplesPerBlock), bm, bound);
        m = fmaxf(m, bm);
    };
#pragma unroll
    for (int u = 0; u < kHeldHeads; ++u) note(held[u]);
    for (int i = (int)threadIdx.x + kHeldHeads * kReduceThreads; i < n_range; i += kReduceThreads) note(segment(b0 + i));
    static_assert(kHeads == 2 * kReduceThreads && kHeldHeads % 2 == 0, "two bounds a thread and chunk");
    auto to_lds = [&] {
        head[threadIdx.x] = held[0];
        head[kReduceThreads + threadIdx.x] = held[1];
#pragma unroll
        for (int u = 2; u < kHeldHeads; ++u) held[u - 2] = held[u];
    };
    to_lds();
    bound = wave_sum(bound);
    m = wave_max(m);
    if ((threadIdx.x & 63) == 63) w_part[threadIdx.x >> 6] = make_float2(bound, m);
    __syncthreads();  // (also orders the cleared accumulators before the additions)
    static_assert(kReduceThreads / 64 == 16, "a wave's partials fill a row");
    const float2 of_wave = w_part[threadIdx.x & 15];
    int ex = 0;
    for (int c0 = b0; c0 < b1; c0 += kHeads) {
        const int n = min(kHeads, b1 - c0);
        if (c0 != b0) {
            if (c0 - b0 < kHeldHeads * kReduceThreads)
                to_lds();
            else
                for (int i = threadIdx.x; i < n; i += kReduceThreads) head[i] = segment(c0 + i);
            __syncthreads();
        }
        // Steps of up to kSegStep * kSegLanes records of one segment: the lane's
        // records are u * kSegLanes < left.  Loads are unconditional, of clamped
        // addresses, and looked at two steps later, so that none waits for
        // another; the steps' registers take turns, for the same reason.
        struct Step {
            uint32_t lo[kSegStep], hi[kSegStep];
            int left, sh0;
            bool any;
        };
        int b = (int)(threadIdx.x / kSegLanes), p = 0, end = 0;
        uint2 h = head[min(b, n - 1)];
        p = (int)(h.x & 0xffffu);
        end = (int)(h.x >> 16);
        auto fetch = [&](Step& st) {
            const int64_t base = (item0 + c0 + min(b, n - 1)) * kRecordsPerBlock;
            st.any = b < n;
            st.left = b < n ? end - p - ln : 0;
            // a record (qx, qy, r) is worth (qx, qy) 2^(sh0 - r); in fixed point
            // that is (qx, qy) 2^(sh0 + ex - r)
            st.sh0 = block_rec_exp(__uint_as_float(h.y)) - (MB - 1);
#pragma unroll
            for (int u = 0; u < kSegStep; ++u) {
                const int i = p + ln + u * kSegLanes;
                // (a segment may be empty and start at the end of the block's range)
                const int64_t at = base + (i < end ? i : min(p, kRecordsPerBlock - 1));
                if constexpr (kCompact) {
                    const uint32_t* words = reinterpret_cast<const uint32_t*>(a.recs);
                    st.lo[u] = words[at];
                    st.hi[u] = reinterpret_cast<const uint16_t*>(words + a.n_records)[at];
                } else {
                    const uint2 w = reinterpret_cast<const uint2*>(a.recs)[at];
                    st.lo[u] = w.x;
                    st.hi[u] = w.y;
                }
            }
            // the next step: the rest of this segment, or the next block's
            p += kSegStep * kSegLanes;
            if (p >= end) {
                b += kSegGroups;
                h = head[min(b, n - 1)];
                p = (int)(h.x & 0xffffu);
                end = (int)(h.x >> 16);
            }
        };
        auto add = [&](const Step& st) {
            const int sh0 = st.sh0 + ex;
#pragma unroll
            for (int u = 0; u < kSegStep; ++u) {
                uint32_t key;
                int r, qx, qy;
                decode_record<EB, MB>(st.lo[u], st.hi[u], key, r, qx, qy);
                if (u * kSegLanes < st.left) {
                    atomicAdd(&acc[key], (unsigned long long)scale_mantissa(qx, sh0 - r));
                    atomicAdd(&acc[kTileRows + key], (unsigned long long)scale_mantissa(qy, sh0 - r));
                }
            }
        };
        Step s0, s1, s2;
        fetch(s0);
        fetch(s1);
        if (c0 == b0)  // (under the first records' loads)
            ex = __builtin_amdgcn_readlane(fixed_point_exp(row_sum(of_wave.x), row_max(of_wave.y)), 15);
        while (s0.any) {
            fetch(s2);
            add(s0);
            if (!s1.any) break;
            fetch(s0);
            add(s1);
            if (!s2.any) break;
            fetch(s1);
            add(s2);
        }
        __syncthreads();
    }
    __syncthreads();
    if (n_split > 1) {
        const int64_t slot = o.part_off + o.part_base[l] + (int64_t)tt * n_split + part;
        unsigned long long* out = a.parts + slot * (2 * kTileRows);
        if (threadIdx.x == 0) a.part_exp[slot] = ex;
        for (int i = threadIdx.x; i < n_rows; i += kReduceThreads) {
            out[i] = acc[i];
            out[kTileRows + i] = acc[kTileRows + i];
        }
        return;
    }
    float2* g = reinterpret_cast<float2*>(a.g_table + o.g_off) + ((int64_t)l << o.grid.log2_table) + row0;
    for (int i = threadIdx.x; i < n_rows; i += kReduceThreads) {
        const long long sx = (long long)acc[i], sy = (long long)acc[kTileRows + i];
        if (sx == 0 && sy == 0) continue;
        float2 w = g[i];
        w.x += (float)ldexp((double)sx, -ex);
        w.y += (float)ldexp((double)sy, -ex);
        g[i] = w;
    }
}

// Tiles reduced in several ranges: the ranges' sums added in FP64, one thread per
// row; blockIdx.y counts the pass's split tiles.
template <bool kMany>
__global__ __launch_bounds__(kCombineThreads) void k_scatter_combine(ScatterArgs a)
{
    const int64_t ct = blockIdx.y;
    const ScatterObj& o = sobj<kMany>(a, last_le<kMany>(a, ct, [](const ScatterObj& v) { return v.ctile_off; }));
    const int cl = (int)(ct - o.ctile_off);
    const int l = level_of(o.ctile_base, o.grid.n_levels, cl);
    const int n_split = o.split[l];
    const int tt = cl - o.ctile_base[l];
    const int64_t row0 = (int64_t)tt << kTileBits;
    const int i = (int)(blockIdx.x * kCombineThreads + threadIdx.x);
    if (i >= (int)min((int64_t)kTileRows, o.level_rows[l] - row0)) return;
    const int64_t slot = o.part_off + o.part_base[l] + (int64_t)tt * n_split;
    const unsigned long long* in = a.parts + slot * (2 * kTileRows) + i;
    double sx = 0.0, sy = 0.0;
#pragma unroll 4
    for (int k = 0; k < n_split; ++k) {
        const double scale = ldexp(1.0, -a.part_exp[slot + k]);
        sx = fma((double)(long long)in[(int64_t)k * 2 * kTileRows], scale, sx);
        sy = fma((double)(long long)in[(int64_t)k * 2 * kTileRows + kTileRows], scale, sy);
    }
    if (sx == 0.0 && sy == 0.0) return;
    float2* g = reinterpret_cast<float2*>(a.g_table + o.g_off) + ((int64_t)l << o.grid.log2_table) + row0;
    float2 w = g[i];
    w.x += (float)sx;
    w.y += (float)sy;
    g[i] = w;
}

template <bool kMany, bool kCompact>
hipError_t place_impl(const ScatterArgs& a, hipStream_t s)
{
    const size_t lds = place_lds_bytes(a.tiles_max, kCompact);
    hipLaunchKernelGGL((k_scatter_place<kMany, kCompact>), dim3((uint32_t)a.n_items), dim3(kPlaceThreads), lds, s, a);
    return hipGetLastError();
}
static_assert(place_lds_bytes(kMaxTilesPerLevel, false) <= 65536, "place LDS");

template <bool kMany>
hipError_t scatter_phase_impl(const ScatterArgs& a, int phase, hipStream_t s)
{
    switch (phase) {
        case 0: return a.compact ? place_impl<kMany, true>(a, s) : place_impl<kMany, false>(a, s);
        case 1:
            if (a.compact)
                hipLaunchKernelGGL((k_scatter_reduce<kMany, true>), dim3((uint32_t)a.n_ritems), dim3(kReduceThreads), 0,
                                   s, a);
            else
                hipLaunchKernelGGL((k_scatter_reduce<kMany, false>), dim3((uint32_t)a.n_ritems), dim3(kReduceThreads), 0,
                                   s, a);
            break;
        case 2:
            hipLaunchKernelGGL(k_scatter_combine<kMany>, dim3(kTileRows / kCombineThreads, (uint32_t)a.n_ctiles),
                               dim3(kCombineThreads), 0, s, a);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

ScatterObj scatter_obj(const GridInfo& g, int64_t n_s)
{
    ScatterObj o{};
    o.grid = g;
    o.n_s = n_s;
    o.n_blocks = (int32_t)((n_s + kSamplesPerBlock - 1) / kSamplesPerBlock);
    o.n_tiles = 0;
    const int64_t T = (int64_t)1 << g.log2_table;
    for (int l = 0; l < g.n_levels; ++l) {
        const int64_t side = (int64_t)g.res[l] + 1;
        const int64_t rows = ((g.dense_mask >> l) & 1u) ? side * side * side : T;
        o.level_rows[l] = rows;
        o.tiles[l] = (int32_t)((rows + kTileRows - 1) / kTileRows);
        o.tile_base[l] = o.n_tiles;
        o.n_tiles += o.tiles[l];
    }
    return o;
}

int64_t scatter_items(const ScatterObj& o) { return (int64_t)o.grid.n_levels * o.n_blocks; }
int64_t scatter_records(const ScatterObj& o) { return scatter_items(o) * kRecordsPerBlock; }
int64_t scatter_segs(const ScatterObj& o) { return (int64_t)o.n_blocks * (o.n_tiles + o.grid.n_levels); }

// Every tile of a level is estimated at an even share of the level's records.
// A tile's ranges are ceil(kReduceItems times its share of the pass, or of
// kReduceItems * kReduceMinRecords records in a smaller pass) in whole numbers:
// with an object alone in its pass the share does not fall when its samples
// grow, so a plan of fewer samples fits the arrays of one of more (rounded
// quotients would ask for one range more whenever they pass an integer).
void scatter_split(ScatterObj& o, int64_t records)
{
    const int64_t pass = records > kReduceItems * kReduceMinRecords ? records : kReduceItems * kReduceMinRecords;
    o.n_ritems = o.n_ctiles = 0;
    o.n_parts = 0;
    for (int l = 0; l < o.grid.n_levels; ++l) {
        const int64_t level = (int64_t)o.n_blocks * kRecordsPerBlock * kReduceItems;  // < 2^43
        int64_t k = (level + o.tiles[l] * pass - 1) / (o.tiles[l] * pass);
        k = k > o.n_blocks ? o.n_blocks : k;
        if (k < 1) k = 1;
        o.split[l] = (int32_t)k;
        o.ritem_base[l] = o.n_ritems;
        o.n_ritems += (int32_t)(o.tiles[l] * k);
        o.part_base[l] = o.n_parts;
        o.ctile_base[l] = o.n_ctiles;
        if (k > 1) {
            o.n_parts += (int32_t)(o.tiles[l] * k);
            o.n_ctiles += o.tiles[l];
        }
    }
}

ScatterObj scatter_plan(const GridInfo& g, int64_t n_s)
{
    ScatterObj o = scatter_obj(g, n_s);
    scatter_split(o, scatter_records(o));
    return o;
}

// A level in k = ceil(x) > 1 ranges a tile has tiles * k < 2 tiles * x parts, and
// the tiles * x of a pass's levels add up to kReduceItems at most.
int64_t scatter_parts_most(int64_t records)
{
    const int64_t full = kReduceItems * kReduceMinRecords;
    return records < full ? 2 * records / kReduceMinRecords : 2 * kReduceItems;
}

size_t scatter_part_bytes() { return sizeof(unsigned long long) * 2 * kTileRows; }

int scatter_tiles_max(const ScatterObj& o)
{
    int m = 1;
    for (int l = 0; l < o.grid.n_levels; ++l) m = o.tiles[l] > m ? o.tiles[l] : m;
    return m;
}

const char* const kScatterPhaseNames[kScatterPhases] = {"k_scatter_place", "k_scatter_reduce", "k_scatter_combine"};

hipError_t launch_scatter_phase(const ScatterArgs& a, int phase, hipStream_t s)
{
    if (a.n_items == 0 || (phase == 2 && a.n_ctiles == 0)) return hipSuccess;
    return a.n_obj == 1 && a.objs == nullptr ? scatter_phase_impl<false>(a, phase, s)
                                             : scatter_phase_impl<true>(a, phase, s);
}

}  // namespace prenom
