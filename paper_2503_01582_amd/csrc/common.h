// Internal declarations shared by the HIP translation units of libprenom.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "prenom.h"

namespace prenom {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
// Compute units of a gfx950 in one partition.  Plans are cut for them, so that they
// are a function of the sizes alone; a device with fewer runs them in more rounds.
constexpr int64_t kCus = 256;

// Level table of a hash grid, passed by value to kernels.
struct GridInfo {
    int32_t res[PRENOM_MAX_LEVELS];
    uint32_t dense_mask;  // bit l set: level l stored 1:1 ((N_l+1)^3 <= T)
    int32_t n_levels;
    int32_t log2_table;
};

// Table row of lattice vertex (vx, vy, vz) on one level: 1:1 on dense levels,
// otherwise the XOR-of-primes spatial hash of the multiresolution hash
// encoding (Mueller et al. 2022) reduced modulo 2^32 and masked to T.
__device__ __forceinline__ uint32_t corner_row(bool dense, uint32_t side, uint32_t log2T, uint32_t vx,
                                               uint32_t vy, uint32_t vz)
{
    if (dense) return vx + side * (vy + side * vz);
    return (vx ^ (vy * 2654435761u) ^ (vz * 805459861u)) & ((1u << log2T) - 1u);
}

// Cell of x on a lattice of resolution N: c = min(floor(x N), N - 1) of the
// exact product, and the local coordinate f = x N - c rounded to FP32.  In
// FP32: N < 2^20 is exact, and rounding x N to nearest never takes it below
// an integer it reaches, so floor of the rounded product is the exact floor
// or one above it; fma(x, N, -c) is the exact x N - c rounded once, so its
// sign tells which, and after the clamp it is f itself.
__device__ __forceinline__ void lattice_cell(float x, int N, uint32_t& c, float& f)
{
    const float Nf = (float)N;
    float cf = floorf(x * Nf);
    if (fmaf(x, Nf, -cf) < 0.0f) cf -= 1.0f;
    cf = fminf(fmaxf(cf, 0.0f), (float)(N - 1));
    c = (uint32_t)cf;
    f = fmaf(x, Nf, -cf);
}

// The 8 cell corners of x on level l: the cell, table rows and trilinear
// weights (corner e = (e & 1, e >> 1 & 1, e >> 2 & 1)).  Used by the forward
// encoding and by the scatter, so they agree bit for bit.
struct Corners {
    uint32_t cell[3];
    uint32_t row[8];
    float w[8];
};

// Sample position in the object frame: clamp(fmaf(t, d, o), 0, 1).
__device__ __forceinline__ float sample_coord(float t, float d, float o)
{
    return fminf(fmaxf(fmaf(t, d, o), 0.0f), 1.0f);
}

template <bool kBranch = false>
__device__ __forceinline__ void level_corners(const GridInfo& g, int l, float x0, float x1, float x2, Corners& c)
{
    const int N = g.res[l];
    const bool dense = (g.dense_mask >> l) & 1u;
    float f[3];
    lattice_cell(x0, N, c.cell[0], f[0]);
    lattice_cell(x1, N, c.cell[1], f[1]);
    lattice_cell(x2, N, c.cell[2], f[2]);
    // Rows of the 8 corners from two products per level (corner_row of each
    // corner, strength-reduced): (c + 1) P = c P + P modulo 2^32 for the hash,
    // and the 1:1 row of a corner is the cell's row plus 1, side or side^2.
    // kBranch: one uniform branch instead of a select per corner (fewer vector
    // instructions, which bind the scatter and the encoding from LDS; the
    // encoding that is bound by its gathers is faster without: 11.4 against 12.2 ms
    // on 48 objects).
    const uint32_t mask = (1u << g.log2_table) - 1u, side = (uint32_t)N + 1u;
    auto dense_row = [&](uint32_t r0, int e) { return r0 + (e & 1) + (e & 2 ? side : 0u) + (e & 4 ? side * side : 0u); };
    auto hash_row = [&](uint32_t hy, uint32_t hz, int e) {
        return ((c.cell[0] + (e & 1)) ^ (e & 2 ? hy + 2654435761u : hy) ^ (e & 4 ? hz + 805459861u : hz)) & mask;
    };
    if constexpr (kBranch) {
        if (dense) {
            const uint32_t r0 = c.cell[0] + side * (c.cell[1] + side * c.cell[2]);
#pragma unroll
            for (int e = 0; e < 8; ++e) c.row[e] = dense_row(r0, e);
        } else {
            const uint32_t hy = c.cell[1] * 2654435761u, hz = c.cell[2] * 805459861u;
#pragma unroll
            for (int e = 0; e < 8; ++e) c.row[e] = hash_row(hy, hz, e);
        }
    } else {
        uint32_t r0 = 0, hy = 0, hz = 0;
        if (dense) {
            r0 = c.cell[0] + side * (c.cell[1] + side * c.cell[2]);
        } else {
            hy = c.cell[1] * 2654435761u;
            hz = c.cell[2] * 805459861u;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) c.row[e] = dense ? dense_row(r0, e) : hash_row(hy, hz, e);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        c.w[e] = (e & 1 ? f[0] : 1.0f - f[0]) * (e & 2 ? f[1] : 1.0f - f[1]) * (e & 4 ? f[2] : 1.0f - f[2]);
}

// ------------------------------------------------------------------ table tiles
// The hash-table gradient buckets contributions by table tile (2^13 rows),
// per (level, block of kScatterBlockSamples samples).
constexpr int kTileBits = 13;
constexpr int kTileRows = 1 << kTileBits;
constexpr int kMaxTilesPerLevel = 1 << (24 - kTileBits);  // T <= 2^24
constexpr int kScatterBlockSamples = 512;
// Place combines the rank atomics of a wave per tile first on levels of at
// most this many tiles, where most lanes of a wave share a tile.  With more
// tiles the leader rounds cost more vector instructions than the LDS
// serialisation of same-address atomics they save, dense levels included
// (48-object place on gfx950: 17.2 ms aggregating up to 16 tiles, 16.3 ms
// up to 4 hashed or 16 dense, 15.7 ms up to 2).
constexpr int kAggregateTiles = 2;

// Adds `unit` to hist[tile] for every active lane and returns the lane's rank
// among the additions to that tile, in units.  Lanes of the wave that share the tile of
// the first remaining lane are combined into one LDS atomic issued by that
// lane (same-address atomics of one instruction would otherwise serialise);
// after kAggregateRounds such rounds the lanes left use plain LDS atomics, so
// a wave spread over many tiles does not pay one round per tile.  Every slot
// comes from an atomic on the same counter, so ranks are distinct whichever
// way a lane takes.
constexpr int kAggregateRounds = 2;

__device__ __forceinline__ uint32_t wave_aggregated_add(uint32_t* hist, uint32_t tile, uint32_t unit)
{
    const int lane = threadIdx.x & 63;
    const uint64_t lane_lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t remaining = __ballot(1);
    uint32_t rank = 0;
    bool placed = false;
#pragma unroll
    for (int round = 0; round < kAggregateRounds; ++round) {
        if (remaining == 0) break;
        const int leader = __ffsll((unsigned long long)remaining) - 1;
        const uint32_t lt = __shfl(tile, leader);
        const uint64_t mask = __ballot(tile == lt);
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(&hist[lt], unit * (uint32_t)__popcll(mask));
        base = __shfl(base, leader);
        if (tile == lt) {
            rank = base + unit * (uint32_t)__popcll(mask & lane_lt);
            placed = true;
        }
        remaining &= ~mask;
    }
    if (!placed) rank = atomicAdd(&hist[tile], unit);
    return rank;
}

// Lane exchange within a row of 16 lanes (DPP): kCtrl = 0x100 + n (row_shl:
// lane i reads lane i + n, 0 past the row end) or 0x110 + n (row_shr: lane i
// reads lane i - n, 0 before the row start).  All lanes must be active.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true);
}

template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}

// Merging repeated cells.  Consecutive samples of a ray often share a cell on
// the coarser levels, so all eight corner rows repeat on neighbouring lanes;
// such a run becomes one record per corner (the sum of its contributions).
// Runs stay inside groups of 8 lanes.  True when the lane starts a run: it has
// a contribution and is the first of its group of 8, or lane - 1 has none or
// another cell.  Every lane of the wave must call it.
__device__ __forceinline__ bool run_head(const Corners& c, bool has)
{
    const uint32_t x = has ? c.cell[0] : 0xffffffffu;  // no lattice coordinate is as large
    const uint32_t other = (dpp_u32<0x111>(x) ^ x) | (dpp_u32<0x111>(c.cell[1]) ^ c.cell[1]) |
                           (dpp_u32<0x111>(c.cell[2]) ^ c.cell[2]);
    return has && ((threadIdx.x & 7) == 0 || other != 0u);
}

// Per lane that starts a run (boundary set): the sums of v over its run (the
// lane and the following lanes of its group of 8 up to the next boundary); a
// segmented suffix scan in three steps, in a fixed order.  Lanes without a
// contribution pass v = 0 and boundary = true; values and their sums have to be
// finite (other runs' are multiplied by 0).  Every lane of the wave must call it.
__device__ __forceinline__ void run_sum(float2 (&v)[8], bool boundary)
{
    const int g = threadIdx.x & 7;
    const int lane = threadIdx.x & 63;
    const uint64_t B = __ballot(boundary);
    // lane + 1 .. lane + d continue this lane's run (they lie in its group)
    const bool c1 = g + 1 < 8 && ((B >> (lane + 1)) & 1ull) == 0;
    const bool c2 = g + 2 < 8 && ((B >> (lane + 1)) & 3ull) == 0;
    const bool c4 = g + 4 < 8 && ((B >> (lane + 1)) & 15ull) == 0;
    // A product with 0 or 1, its addition and the lane exchange are one
    // instruction (v_fmac with a DPP operand), a third of what an exchange, a
    // select and an addition take.  An exchanged operand may be read two
    // instructions after it was written: the 16 values of a step lie between.
    const float m1 = c1 ? 1.0f : 0.0f, m2 = c2 ? 1.0f : 0.0f, m4 = c4 ? 1.0f : 0.0f;
#define PRENOM_RUN1(i, m, n) "v_fmac_f32_dpp %" #i ", %" #i ", %" #m " row_shl:" #n " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
#define PRENOM_RUN16(m, n)                                                                                    \
    PRENOM_RUN1(0, m, n) PRENOM_RUN1(1, m, n) PRENOM_RUN1(2, m, n) PRENOM_RUN1(3, m, n) PRENOM_RUN1(4, m, n)   \
    PRENOM_RUN1(5, m, n) PRENOM_RUN1(6, m, n) PRENOM_RUN1(7, m, n) PRENOM_RUN1(8, m, n) PRENOM_RUN1(9, m, n)   \
    PRENOM_RUN1(10, m, n) PRENOM_RUN1(11, m, n) PRENOM_RUN1(12, m, n) PRENOM_RUN1(13, m, n)                    \
    PRENOM_RUN1(14, m, n) PRENOM_RUN1(15, m, n)
    asm("s_nop 4\n\t" PRENOM_RUN16(16, 1) PRENOM_RUN16(17, 2) PRENOM_RUN16(18, 4) "s_nop 1"
        : "+v"(v[0].x), "+v"(v[0].y), "+v"(v[1].x), "+v"(v[1].y), "+v"(v[2].x), "+v"(v[2].y), "+v"(v[3].x),
          "+v"(v[3].y), "+v"(v[4].x), "+v"(v[4].y), "+v"(v[5].x), "+v"(v[5].y), "+v"(v[6].x), "+v"(v[6].y),
          "+v"(v[7].x), "+v"(v[7].y)
        : "v"(m1), "v"(m2), "v"(m4));
#undef PRENOM_RUN16
#undef PRENOM_RUN1
}

// ------------------------------------------------------------------ batches
// Device descriptor of one object of a batch (offsets index the batch's
// concatenated arrays; objects own consecutive rays).
struct ObjDev {
    GridInfo grid;
    int32_t table_dtype;  // PRENOM_F32 or PRENOM_F16 (read the FP16 parameter copy)
    int32_t prior_res;
    int32_t pad_[2];
    int64_t param_off;    // floats: first parameter (the tables) of the object
    int64_t ray_begin, n_rays;
    int64_t y_off;        // floats: the object's features [L][n_s][2] (and their gradient)
    const float* prior;   // [R^3] or null (uniform sampling)
    double A[12];         // world -> object frame
};

// Object of a batch that holds ray `ray` (objects are contiguous in rays).
__device__ __forceinline__ int find_object(const ObjDev* objs, int n_obj, int64_t ray)
{
    int lo = 0, hi = n_obj - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (objs[mid].ray_begin <= ray)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// ------------------------------------------------------------------ XCD order
// Item of a block of a launch whose items should stay on one XCD in runs: blocks go to
// the 8 XCDs in turn, and each XCD's L2 fetches what its blocks read.
constexpr uint32_t kXcds = 8;

__host__ __device__ __forceinline__ uint32_t xcd_item(uint32_t block, int run_log2)
{
    const uint32_t slot = block / kXcds, xcd = block % kXcds;
    return ((slot >> run_log2) * kXcds + xcd) << run_log2 | (slot & ((1u << run_log2) - 1u));
}

int xcd_run_log2(int64_t n_items);

// ------------------------------------------------------------------ launches
// Every launcher returns hipSuccess or the launch error.

struct SampleArgs {
    int32_t n_coarse, n_fine, include_coarse, use_prior;
    double eps, near_t, far_t;
    double A[12];
    const float* prior;
    int32_t R;
    const float* rays_o;
    const float* rays_d;
    const float* xi;
    int64_t n;
    float* ray_obj;
    float* t;
    float* dt;
    int32_t* bins;
    uint8_t* flags;
};
hipError_t launch_sample(const SampleArgs& a, hipStream_t s);
hipError_t launch_sample_batch(const SampleArgs& a, const ObjDev* objs, int n_obj, hipStream_t s);

// Encoding of the grid vertices p0 .. p0 + cnt - 1 of the R^3 grid, vertex
// p = (k R + j) R + i at (i, j, k) / (R - 1): features [L][cnt][2]; and the
// density column of head outputs sc [n][4] into out [n].
hipError_t launch_encode_grid(const GridInfo& g, const float* table, const void* table_f16, int32_t R, int64_t p0,
                              int64_t cnt, float* y, hipStream_t s);
hipError_t launch_density_grid(const float* sc, int64_t n, float* out, hipStream_t s);

// Encoding of explicit positions: features [L][n][2], optional corner rows.
hipError_t launch_encode_points(const GridInfo& g, const float* table, const float* pos, int64_t n,
                                float* features, int32_t* corner_idx, hipStream_t s);

struct ScatterObj;
// Encoding of the rendered samples of every object of a batch (FP16 tables come
// from params_f16).  encode_split shares the objects between the kernel that
// stages tables in LDS (lds_off, n_runs, run of sobjs) and the one block per
// (level, sample block) of the others (item_off); n_lds, n_items: their blocks.
void encode_split(const ObjDev* objs, ScatterObj* sobjs, int n_obj, int64_t& n_items, int64_t& n_lds);
hipError_t launch_encode_batch(const ObjDev* objs, const ScatterObj* sobjs, int n_obj, int64_t n_items, int64_t n_lds,
                               const float* params, const void* params_f16, const float* ray_obj, const float* t,
                               int32_t S, float* y, hipStream_t s);

// Encoding of the rendered samples (positions from rays and t); reads the
// FP16 table copy when table_f16 is not null, the FP32 tables otherwise.
hipError_t launch_encode_samples(const GridInfo& g, const float* table, const void* table_f16,
                                 const float* ray_obj, const float* t, int64_t n_rays, int32_t S, float* y,
                                 hipStream_t s);

// Bucketed scatter-add of the feature gradients into the table gradient.
// Geometry of one object's scatter: its table tiles and sample blocks, and
// where its pieces sit in the (possibly batched) arrays.
struct ScatterObj {
    GridInfo grid;
    int32_t n_blocks;  // sample blocks per level
    int32_t n_tiles;   // table tiles over the object's levels
    int32_t n_ritems;  // reduce items
    int32_t n_ctiles;  // tiles reduced in several ranges of blocks
    int32_t n_parts;   // 64-bit partial sums of those (one per range)
    int32_t tiles[PRENOM_MAX_LEVELS];
    int32_t tile_base[PRENOM_MAX_LEVELS];
    int32_t split[PRENOM_MAX_LEVELS];       // ranges of blocks each of the level's tiles is reduced in
    int32_t ritem_base[PRENOM_MAX_LEVELS];  // the level's first reduce item (tile-major, then range)
    int32_t part_base[PRENOM_MAX_LEVELS];   // its first partial sum, and
    int32_t ctile_base[PRENOM_MAX_LEVELS];  // its first split tile (where split > 1)
    int64_t level_rows[PRENOM_MAX_LEVELS];
    int64_t n_s;        // samples
    int64_t s_begin;    // first sample in the per-sample arrays (t; ray = sample / S)
    int64_t dy_off;     // float2 index of the object's dy [L][n_s]
    int64_t g_off;      // float index of the object's table gradient
    int64_t item_off;   // first (level, sample block) item
    int64_t seg_off;    // first entry of its segment starts
    int64_t ritem_off;  // first reduce item
    int64_t part_off;   // first partial sum
    int64_t ctile_off;  // first split tile
    int64_t lds_off;    // staged encoding: first (level, run) block,
    int64_t run;        // samples per run, and
    int32_t n_runs;     // runs per level (0: not staged)
};
// Fills the geometry of one object (offsets within the batch are left 0).
ScatterObj scatter_obj(const GridInfo& g, int64_t n_s);
int64_t scatter_items(const ScatterObj& o);      // L * n_blocks
int64_t scatter_records(const ScatterObj& o);    // record capacity: 4096 per item
int64_t scatter_segs(const ScatterObj& o);       // segment starts
int scatter_tiles_max(const ScatterObj& o);      // max tiles of one level
// The object's split of its tiles into reduce items, in a pass over `records`
// of capacity.
void scatter_split(ScatterObj& o, int64_t records);
// Geometry of an object in a pass of its own; no array of it grows when n_s falls.
ScatterObj scatter_plan(const GridInfo& g, int64_t n_s);
// Partial sums that a pass over `records` needs at most, however they are spread
// over objects and levels.
int64_t scatter_parts_most(int64_t records);
size_t scatter_part_bytes();                     // one partial sum

struct ScatterArgs {
    int32_t S;
    float inv_S;                // 1 / S
    int32_t n_obj;              // 1: `one` holds the object; else `objs` (device) holds n_obj of them
    int32_t tiles_max;          // max tiles of one level over all objects
    int64_t n_items;            // (object, level, sample block) items
    int64_t n_ritems;           // reduce items
    int64_t n_ctiles;           // tiles reduced in several ranges
    ScatterObj one;
    const ScatterObj* objs;
    const float* ray_obj;
    const float* t;
    const float2* dy;
    float* g_table;
    float* block_max;           // [n_items] max |dy| of the item
    uint16_t* seg;              // per item [tiles + 1]: start of each tile's segment, and the end
    unsigned long long* parts;  // partial sums: 64-bit fixed point, [2][tile rows] each, and
    int32_t* part_exp;          // their exponents
    uint64_t* recs;             // packed records (scatter.hip), 4096 per item
    int64_t n_records;          // length of recs
    int32_t* nonfinite;         // set to 1 when a dy entry is not finite (loss scaling), or null
    // 1: compact records (15-bit mantissas, 48 bits: 32-bit words at recs,
    // then n_records 16-bit words), for FP16 tables; 0: 64-bit records.
    int32_t compact;
};
// The scatter runs as kScatterPhases dependent kernels, launched in order:
// place, reduce, combine (none where no tile is split).
constexpr int kScatterPhases = 3;
extern const char* const kScatterPhaseNames[kScatterPhases];
hipError_t launch_scatter_phase(const ScatterArgs& a, int phase, hipStream_t s);

// MLP: forward writes (sigma, r, g, b) per sample; backward recomputes the
// activations, writes dy and per-block partial weight gradients.
struct MlpShape {
    int32_t in_dim, width, hidden, dtype;
};
bool mlp_supported(const MlpShape& m);

// One block's share of a batched MLP launch: tiles [tile_begin, tile_end) of
// one object.  w_off (floats) locates the object's MLP weights in the batch
// parameters, y_off (floats) its features (level-major [L][n_s][2]), s_off
// (samples) its first sample in the per-sample arrays, a_off (floats) its
// stored activations and deltas when the MLP is 128 wide and FP32.
struct MlpWork {
    int64_t w_off, y_off, s_off, n_s;
    int64_t tile_begin, tile_end;
    int64_t a_off;
};

// The 128-wide FP32 MLP stores its hidden activations in the forward and runs
// its backward as a chain kernel (deltas, dy) and a weight-gradient kernel; the
// two buffers hold act[D][n_s][W] and delta[D][n_s][W].  The 16-bit form
// recomputes them in one kernel.
constexpr int kWideWidth = 128;
inline int64_t mlp_act_floats(const MlpShape& m, int64_t n_s)
{
    return m.width >= kWideWidth && m.dtype == PRENOM_F32 ? 2 * (int64_t)m.hidden * n_s * m.width : 0;
}
int mlp_bwd_waves(int64_t n_samples);  // partial-gradient slots (one per block) the bwd writes
// act: activation/delta buffer of mlp_act_floats floats (128-wide FP32 MLPs; else unused)
hipError_t launch_mlp_fwd(const MlpShape& m, const float* w, const float* y, int64_t n_s, float* sc, float* act,
                          hipStream_t s);
hipError_t launch_mlp_bwd(const MlpShape& m, const float* w, const float* y, const float* dout, const float* sc,
                          int64_t n_s, float* dy, float* partial, float* act, hipStream_t s);
hipError_t launch_mlp_fwd_lp(const MlpShape& m, const float* w, const float* y, int64_t n_s, float* sc,
                             hipStream_t s);
hipError_t launch_mlp_bwd_lp(const MlpShape& m, const float* w, const float* y, const float* dout, const float* sc,
                             int64_t n_s, float* dy, float* partial, hipStream_t s);
hipError_t launch_mlp_fwd_batch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params,
                                const float* y, float* sc, float* act, hipStream_t s);
// chain: the runs in which the 128-wide backward computes deltas and dy (any split).
hipError_t launch_mlp_bwd_batch(const MlpShape& m, const MlpWork* work, int n_blocks, const MlpWork* chain,
                                int n_chain, const float* params, const float* y, const float* dout, const float* sc, float* dy, float* partial,
                                int64_t slot_stride, float* act, hipStream_t s);
hipError_t launch_mlp_fwd_lp_batch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params,
                                   const float* y, float* sc, hipStream_t s);
hipError_t launch_mlp_bwd_lp_batch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params,
                                   const float* y, const float* dout, const float* sc, float* dy, float* partial,
                                   int64_t slot_stride, hipStream_t s);
hipError_t launch_reduce_partials(const float* partial, int n_slots, int64_t n_mlp, float* g_mlp,
                                  hipStream_t s);

// Per object of a batch: where its backward partials sit and where its MLP
// gradient goes.  mlp_begin is the prefix of n_mlp over the objects.
struct MlpRed {
    int64_t mlp_begin, n_mlp;
    int64_t partial_off;  // floats
    int64_t n_slots;      // partials (each n_mlp floats, consecutive)
    int64_t g_off;        // floats: the object's MLP gradient in the batch gradient
};
hipError_t launch_reduce_partials_batch(const MlpRed* reds, int n_obj, int64_t n_mlp_total, const float* partial,
                                        float* grads, hipStream_t s);

// Compositing and loss.
struct CompositeArgs {
    int64_t n_rays;
    int64_t norm_rays;    // single object: rays the loss is averaged over (0: n_rays), for calls over a part of them
    int32_t S;
    int32_t loss_mode;
    float lambda_d, lambda_sigma;
    const float* sc;      // [n_s][4]
    const float* t;       // [n_rays][S]
    const float* dt;      // [n_rays][S]
    const uint8_t* flags;
    const float* bg;      // [n][3] or null
    const float* tgt_rgb; // [n][3] or null
    const float* tgt_depth;
    const uint8_t* mask;
    float* rgb;           // fwd outputs, or null (then only ray_state is written)
    float* depth;
    float* opacity;
    float* ray_state;     // [n][8]: rgb(3), depth, T_S, sigma sum, -, -
    double* loss_partial; // [blocks]
    const ObjDev* objs;   // batch: per-object loss normalisation (n = the object's rays), or null
    int32_t n_obj;
    double* ray_loss;     // batch fwd: [n_rays] loss term of each ray
    const float* d_rgb;   // bwd only
    const float* d_depth;
    const float* d_opacity;
    const float* loss_scale;  // bwd: device scalar multiplying the upstream gradient, or null
    float* dout;          // bwd: [n_s][4] (dsigma, dr, dg, db)
};
int composite_loss_blocks(int64_t n_rays);
int composite_rays_per_block();  // rays of one compositing block (its loss partial)
hipError_t launch_composite_fwd(const CompositeArgs& a, hipStream_t s);
hipError_t launch_loss_finalize(const double* partial, int n_blocks, float* loss, hipStream_t s);
hipError_t launch_composite_bwd(const CompositeArgs& a, hipStream_t s);
// loss[o] = sum of ray_loss over the rays of object o (FP64), one block per object.
hipError_t launch_loss_objects(const ObjDev* objs, int n_obj, const double* ray_loss, float* loss, hipStream_t s);

struct AdamArgs {
    float* p;
    float* g;
    float* m;
    float* v;
    int64_t n;
    float lr, beta1, beta2, eps, inv_c1, inv_c2;
    void* table_f16;         // FP16 copy of the first n_table entries, or null
    int64_t n_table;
    float* loss_scale;       // null: plain Adam
    int32_t* scaler_state;   // [2] non-finite flag, finite steps since the last scale change
    int32_t growth_interval;
    int64_t* step_dev;       // non-null: bias corrections from this device step counter, which is
                             // advanced after every applied (not skipped) step
};
hipError_t launch_adam(const AdamArgs& a, hipStream_t s);
// Plain gradient descent p -= lr g on the same arguments (m, v, beta1, beta2,
// eps and the bias corrections unused).
hipError_t launch_sgd(const AdamArgs& a, hipStream_t s);
hipError_t launch_to_f16(const float* src, void* dst, int64_t n, hipStream_t s);

// Reptile's outer update over n_tasks parameter vectors trained from theta:
// theta += beta * mean_b(task_b - theta), then every task slot (and its FP16
// copy, and its Adam moments, when given) restarts from the new theta.
struct ReptileArgs {
    float* theta;
    float* tasks;            // task b at tasks + b * stride
    float* m;                // Adam moments in the task layout, or null
    float* v;
    void* tasks_f16;         // FP16 copy in the task layout (its first n_f16 entries), or null
    int64_t* step;           // device step counter reset to 0, or null
    int64_t n, stride;       // stride a multiple of 4
    int64_t n_f16;
    int32_t n_tasks;
    float beta;
};
hipError_t launch_reptile(const ReptileArgs& a, hipStream_t s);

// Trilinear, vertex-aligned lookup of a density grid F [R][R][R] (x fastest;
// value F[i] at i/(R-1)), each coordinate clamped to [0, 1] (NaN to 0); FP64
// without contraction, the sampler's prior lookup (Eq. (4)) and the canonical
// yaw score (Eq. (3)).
__device__ inline double prior_at(const float* __restrict__ F, int R, const double xin[3])
{
#pragma clang fp contract(off)
    int i0[3];
    double f[3];
    for (int a = 0; a < 3; ++a) {
        double x = xin[a];
        x = x >= 0.0 ? x : 0.0;  // also maps NaN to 0
        x = x > 1.0 ? 1.0 : x;
        const double g = x * (double)(R - 1);
        int i = (int)floor(g);
        i = i > R - 2 ? R - 2 : i;
        i0[a] = i;
        f[a] = g - (double)i;
    }
    double s = 0.0;
#pragma unroll
    for (int cz = 0; cz < 2; ++cz)
#pragma unroll
        for (int cy = 0; cy < 2; ++cy)
#pragma unroll
            for (int cx = 0; cx < 2; ++cx) {
                const double wx = cx ? f[0] : 1.0 - f[0];
                const double wy = cy ? f[1] : 1.0 - f[1];
                const double wz = cz ? f[2] : 1.0 - f[2];
                const double w = wx * wy * wz;
                const int64_t idx = (int64_t)(i0[0] + cx) +
                                    (int64_t)R * ((int64_t)(i0[1] + cy) + (int64_t)R * (i0[2] + cz));
                s += w * (double)F[idx];
            }
    return s;
}

// Canonical yaw search (Eq. (3)).  yaw_split sets the split of a.n points and
// a.K yaws; workspace: per (chunk, yaw) sums, per (extent chunk, yaw) extents.
struct YawArgs {
    const float* pts;   // [n][3]
    int64_t n;
    const float* F;     // [R][R][R]
    int32_t R, K;
    int32_t log2_kl;             // yaws per wave
    int64_t chunk, n_chunks;     // points per score block
    int64_t ext_chunk, n_ext;    // points per extents block
    double2* turn;      // [K] cos, sin
    double* part_sum;   // [n_chunks][K]
    double* part_ext;   // [n_ext + 1][4][K]: min x, min y, max x, max y
    double* part_z;     // [n_ext + 1][2]: min z, max z
    double* scores;     // [K]
    double* extents;    // [K][3]
    double* centers;    // [K][3]
    int32_t* best;
};
void yaw_split(YawArgs& a);
size_t yaw_doubles(const YawArgs& a);
size_t yaw_doubles_most(int64_t n, int64_t K);  // of any call of up to n points and K yaws
void yaw_place(YawArgs& a, double* ws);
hipError_t launch_canonical_yaw(YawArgs a, hipStream_t s);

}  // namespace prenom
