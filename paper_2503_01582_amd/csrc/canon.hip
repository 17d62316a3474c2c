// Canonical yaw search (Sec. III-B, "Object State Canonicalization",
// Eq. (3)).  An object stands on the ground (z up), so its pose in the
// category's canonical frame is searched over the yaw alone: for each of K
// yaws gamma_k = 2 pi k / K the cloud is turned about z, normalised into the
// unit cube by the midpoint and size of its extents (an axis of zero extent
// maps to 1/2), and scored by the sum of the prior's trilinear density over
// its points; the first yaw of largest score wins.
//
// K x |P| lookups of a grid that sits in L2.  A lane is a yaw and walks the
// points: one point's position at neighbouring yaws lies on an arc of the grid,
// so a wave's gather touches the few lines of that arc (with a lane per point
// it touched one line a lane), a point's z cell is found once for all yaws, the
// sums and extents stay in registers to the end, and a sine and cosine serve a
// whole chunk of points.  8927 points x 360 yaws on a 64^3 grid 73 -> 38 us,
// 60000 x 720 682 -> 190, 2^20 x 360 5.74 -> 1.56 ms; the long clouds are bound by
// the gathers (156 cycles of a CU for 64 densities, a quarter of it arithmetic),
// the short ones by the launches and a block's joins.  Three launches:
//   extents : per (point chunk, yaw) the min and max of the turned points
//   score   : per (point chunk, yaw) the density sum; each block first joins
//             the chunks' extents of its yaws (above kYawJoin chunks a launch
//             of its own does)
//   finish  : per yaw the chunk sums added; the first maximum
// FP64 throughout, the turn without contraction; every sum has a fixed order,
// so the result does not depend on scheduling.
#include "common.h"

#pragma clang fp contract(off)

namespace prenom {
namespace {

constexpr int kYawThreads = 256;
constexpr int kYawWaves = kYawThreads / 64;
constexpr int kYawJoin = 32;  // chunks of extents that a score block joins itself
constexpr double kPi = 3.14159265358979323846;

// A wave holds kl yaws (a power of two) and 64 / kl points at a time.
struct Lane {
    int lane, wave, kl, sub, k;  // k: this lane's yaw, clamped to the last
    bool owns;                   // writes the results of its yaw
    __device__ Lane(const YawArgs& a)
        : lane(threadIdx.x & 63), wave(threadIdx.x >> 6), kl(1 << a.log2_kl)
    {
        sub = lane >> a.log2_kl;
        const int g = (int)blockIdx.y * kl + (lane & (kl - 1));
        owns = sub == 0 && g < a.K;
        k = g < a.K ? g : a.K - 1;
    }
};

__device__ __forceinline__ void yaw_rotation(int k, int K, double& c, double& s)
{
    const double g = 2.0 * kPi * (double)k / (double)K;
    c = cos(g);
    s = sin(g);
}

__device__ __forceinline__ double wave_min(double v)
{
    for (int d = 32; d >= 1; d >>= 1) v = fmin(v, __shfl_xor(v, d));
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
    for (int d = 32; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d));
    return v;
}

struct Extent {
    double v[4] = {INFINITY, INFINITY, -INFINITY, -INFINITY};  // min x, min y, max x, max y
    __device__ void add(double x, double y)
    {
        v[0] = fmin(v[0], x);
        v[1] = fmin(v[1], y);
        v[2] = fmax(v[2], x);
        v[3] = fmax(v[3], y);
    }
    __device__ void join(const double o[4])
    {
        v[0] = fmin(v[0], o[0]);
        v[1] = fmin(v[1], o[1]);
        v[2] = fmax(v[2], o[2]);
        v[3] = fmax(v[3], o[3]);
    }
};

// The block's waves join their lanes' extents and z bounds; every wave gets the result.
__device__ __forceinline__ void join_waves(Extent& e, double& zlo, double& zhi, const Lane& L,
                                           double (*red)[4][64], double (*redz)[2])
{
    for (int i = 0; i < 4; ++i) red[L.wave][i][L.lane] = e.v[i];
    if (L.lane == 0) {
        redz[L.wave][0] = zlo;
        redz[L.wave][1] = zhi;
    }
    __syncthreads();
    const int waves = blockDim.x >> 6;
    for (int w = 0; w < waves; ++w) {
        double o[4];
        for (int i = 0; i < 4; ++i) o[i] = red[w][i][L.lane];
        e.join(o);
        zlo = fmin(zlo, redz[w][0]);
        zhi = fmax(zhi, redz[w][1]);
    }
}

// Extents of all chunks of the lane's yaw, and of z: the block's waves and their
// sub lanes take chunks in turn.
__device__ __forceinline__ void join_chunks(const YawArgs& a, const Lane& L, Extent& e, double& zlo, double& zhi)
{
    const int per = 64 >> a.log2_kl, step = per * (int)(blockDim.x >> 6);
#pragma unroll 4
    for (int64_t c = L.wave * per + L.sub; c < a.n_ext; c += step) {
        double o[4];
        for (int i = 0; i < 4; ++i) o[i] = a.part_ext[(4 * c + i) * a.K + L.k];
        e.join(o);
        zlo = fmin(zlo, a.part_z[2 * c]);
        zhi = fmax(zhi, a.part_z[2 * c + 1]);
    }
    for (int d = L.kl; d < 64; d <<= 1) {
        double o[4];
        for (int i = 0; i < 4; ++i) o[i] = __shfl_xor(e.v[i], d);
        e.join(o);
        zlo = fmin(zlo, __shfl_xor(zlo, d));
        zhi = fmax(zhi, __shfl_xor(zhi, d));
    }
}

__global__ __launch_bounds__(kYawThreads) void k_yaw_extents(YawArgs a)
{
    __shared__ double2 pt[kYawThreads];
    __shared__ double red[kYawWaves][4][64], redz[kYawWaves][2];
    const Lane L(a);
    const int64_t c0 = (int64_t)blockIdx.x * a.ext_chunk;
    const int64_t c1 = c0 + a.ext_chunk < a.n ? c0 + a.ext_chunk : a.n;
    double cs, sn;
    yaw_rotation(L.k, a.K, cs, sn);
    Extent e;
    double zlo = INFINITY, zhi = -INFINITY;
    const int per = 64 >> a.log2_kl;
    for (int64_t j0 = c0; j0 < c1; j0 += kYawThreads) {
        const int m = (int)(c1 - j0 < kYawThreads ? c1 - j0 : kYawThreads);
        __syncthreads();
        if ((int)threadIdx.x < m) {
            const float* p = a.pts + 3 * (j0 + threadIdx.x);
            pt[threadIdx.x] = {(double)p[0], (double)p[1]};
            zlo = fmin(zlo, (double)p[2]);
            zhi = fmax(zhi, (double)p[2]);
        }
        __syncthreads();
#pragma unroll 4
        for (int i = L.wave * per + L.sub; i < m; i += kYawWaves * per) {
            const double2 p = pt[i];
            e.add(cs * p.x - sn * p.y, sn * p.x + cs * p.y);
        }
    }
    for (int d = L.kl; d < 64; d <<= 1) {
        double o[4];
        for (int i = 0; i < 4; ++i) o[i] = __shfl_xor(e.v[i], d);
        e.join(o);
    }
    zlo = wave_min(zlo);
    zhi = wave_max(zhi);
    join_waves(e, zlo, zhi, L, red, redz);
    if (L.wave == 0 && L.owns)
        for (int i = 0; i < 4; ++i) a.part_ext[(4 * (int64_t)blockIdx.x + i) * a.K + L.k] = e.v[i];
    if (blockIdx.x == 0 && L.wave == 0 && L.owns) a.turn[L.k] = {cs, sn};
    if (threadIdx.x == 0 && blockIdx.y == 0) {
        a.part_z[2 * blockIdx.x] = zlo;
        a.part_z[2 * blockIdx.x + 1] = zhi;
    }
}

// All chunks' extents into one, for clouds of many chunks.
__global__ __launch_bounds__(1024) void k_yaw_join(YawArgs a, double* __restrict__ ext, double* __restrict__ z)
{
    __shared__ double red[16][4][64], redz[16][2];
    const Lane L(a);
    Extent e;
    double zlo = INFINITY, zhi = -INFINITY;
    join_chunks(a, L, e, zlo, zhi);
    join_waves(e, zlo, zhi, L, red, redz);
    if (L.wave == 0 && L.owns)
        for (int i = 0; i < 4; ++i) ext[(int64_t)i * a.K + L.k] = e.v[i];
    if (threadIdx.x == 0 && blockIdx.y == 0) {
        z[0] = zlo;
        z[1] = zhi;
    }
}

// S = max - min, C = (max + min) / 2 of an axis, and 1 / S; an axis without
// extent maps to 1/2.
struct Axis {
    double S, C, r;
    bool ok;
    __device__ Axis(double lo, double hi) : S(hi - lo), C(0.5 * (hi + lo)), ok(S > 0.0) { r = 1.0 / S; }
    // The point's cell i and place f in it on a grid of R vertices; the lookup's clamps.
    __device__ void cell(double q, int R, int& i, double& f) const
    {
        double x = ok ? fma(q - C, r, 0.5) : 0.5;
        x = x >= 0.0 ? x : 0.0;  // also maps NaN to 0
        x = x > 1.0 ? 1.0 : x;
        const double g = x * (double)(R - 1);
        i = (int)g;  // g >= 0
        i = i > R - 2 ? R - 2 : i;
        f = g - (double)i;
    }
};

__device__ __forceinline__ double mix(double a, double b, double f) { return fma(f, b, (1.0 - f) * a); }

struct YawPoint {
    double x, y, fz;
    int64_t plane;  // element of F where the point's z cell begins
};

__device__ __forceinline__ double yaw_density(const float* __restrict__ F, int R, const YawPoint& p, double cs,
                                              double sn, const Axis& ax, const Axis& ay)
{
    int ix, iy;
    double fx, fy;
    ax.cell(cs * p.x - sn * p.y, R, ix, fx);
    ay.cell(sn * p.x + cs * p.y, R, iy, fy);
    const float* f = F + p.plane;
    const int row = ix + R * iy, up = R * R;
    float2 v[4];
    __builtin_memcpy(&v[0], f + row, 8);
    __builtin_memcpy(&v[1], f + row + R, 8);
    __builtin_memcpy(&v[2], f + row + up, 8);
    __builtin_memcpy(&v[3], f + row + up + R, 8);
    double r[4];
    for (int i = 0; i < 4; ++i) r[i] = mix((double)v[i].x, (double)v[i].y, fx);
    return mix(mix(r[0], r[1], fy), mix(r[2], r[3], fy), p.fz);
}

__global__ __launch_bounds__(kYawThreads) void k_yaw_score(YawArgs a)
{
    __shared__ YawPoint pt[kYawThreads];
    __shared__ double red[kYawWaves][4][64], redz[kYawWaves][2];
    const Lane L(a);
    Extent e;
    double zlo = INFINITY, zhi = -INFINITY;
    join_chunks(a, L, e, zlo, zhi);
    join_waves(e, zlo, zhi, L, red, redz);
    const Axis ax(e.v[0], e.v[2]), ay(e.v[1], e.v[3]), az(zlo, zhi);
    if (blockIdx.x == 0 && L.wave == 0 && L.owns) {
        double* S = a.extents + 3 * (int64_t)L.k;
        double* C = a.centers + 3 * (int64_t)L.k;
        S[0] = ax.S;
        S[1] = ay.S;
        S[2] = az.S;
        C[0] = ax.C;
        C[1] = ay.C;
        C[2] = az.C;
    }
    const double cs = a.turn[L.k].x, sn = a.turn[L.k].y;
    const int64_t c0 = (int64_t)blockIdx.x * a.chunk;
    const int64_t c1 = c0 + a.chunk < a.n ? c0 + a.chunk : a.n;
    const int per = 64 >> a.log2_kl;
    double sum = 0.0;
    for (int64_t j0 = c0; j0 < c1; j0 += kYawThreads) {
        const int m = (int)(c1 - j0 < kYawThreads ? c1 - j0 : kYawThreads);
        __syncthreads();
        if ((int)threadIdx.x < m) {
            const float* p = a.pts + 3 * (j0 + threadIdx.x);
            YawPoint q;
            int iz;
            q.x = p[0];
            q.y = p[1];
            az.cell((double)p[2], a.R, iz, q.fz);
            q.plane = (int64_t)iz * a.R * a.R;
            pt[threadIdx.x] = q;
        }
        __syncthreads();
#pragma unroll 4
        for (int i = L.wave * per + L.sub; i < m; i += kYawWaves * per)
            sum += yaw_density(a.F, a.R, pt[i], cs, sn, ax, ay);
    }
    for (int d = L.kl; d < 64; d <<= 1) sum += __shfl_xor(sum, d);
    __syncthreads();
    red[L.wave][0][L.lane] = sum;
    __syncthreads();
    if (L.wave == 0 && L.owns) {
        double t = sum;
        for (int w = 1; w < kYawWaves; ++w) t += red[w][0][L.lane];
        a.part_sum[(int64_t)blockIdx.x * a.K + L.k] = t;
    }
}

// One block: the chunk sums of each yaw, then the first index of the largest.
// kf lanes hold a yaw each, the wave's other lanes and 16 / groups waves share
// the chunks of a group of kf yaws.
__global__ __launch_bounds__(1024) void k_yaw_finish(YawArgs a, int log2_kf)
{
    __shared__ double part[16][64];
    __shared__ double best_v[16];
    __shared__ int best_k[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kf = 1 << log2_kf, sub = lane >> log2_kf, per = 64 >> log2_kf;
    const int groups = (a.K + kf - 1) >> log2_kf;
    const int slices = groups >= 16 ? 1 : 16 / groups, side = 16 / slices;  // groups summed at a time
    double bv = -INFINITY;
    int bk = 0x7fffffff;
    for (int g0 = 0; g0 < groups; g0 += side) {
        const int slice = wave / side, k = kf * (g0 + wave % side) + (lane & (kf - 1));
        double t = 0.0;
        if (slice < slices && k < a.K) {
#pragma unroll 16
            for (int64_t c = slice * per + sub; c < a.n_chunks; c += slices * per) t += a.part_sum[c * a.K + k];
        }
        for (int d = kf; d < 64; d <<= 1) t += __shfl_xor(t, d);
        __syncthreads();
        part[wave][lane] = t;
        __syncthreads();
        if (slice == 0 && sub == 0 && k < a.K) {
            for (int s = 1; s < slices; ++s) t += part[wave + s * side][lane];
            a.scores[k] = t;
            if (t > bv || (t == bv && k < bk)) {
                bv = t;
                bk = k;
            }
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        const double ov = __shfl_xor(bv, d);
        const int ok = __shfl_xor(bk, d);
        if (ov > bv || (ov == bv && ok < bk)) {
            bv = ov;
            bk = ok;
        }
    }
    if (lane == 0) {
        best_v[wave] = bv;
        best_k[wave] = bk;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 16; ++i)
            if (best_v[i] > bv || (best_v[i] == bv && best_k[i] < bk)) {
                bv = best_v[i];
                bk = best_k[i];
            }
        // every score -inf or NaN: the first yaw, as a sequential first-maximum scan gives
        *a.best = bk == 0x7fffffff ? 0 : bk;
    }
}

int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

// How a call's points and yaws are split over lanes and blocks.
void yaw_split(YawArgs& a)
{
    // Yaws a wave holds: the most that leave less than a seventh of the lanes
    // without one, since neighbouring yaws read neighbouring cells.
    a.log2_kl = 6;
    while (a.log2_kl > 0 && 7 * div_up(a.K, 1 << a.log2_kl) * (1 << a.log2_kl) > 8 * (int64_t)a.K) --a.log2_kl;
    const int64_t groups = div_up(a.K, 1 << a.log2_kl);
    // Two blocks a CU, and four where their chunks are long; no chunk under 32
    // points (a block's joins are paid per chunk) and none above 4096 (the length
    // of a lane's sum).  8927 points x 360 yaws: 37 us with two, 43 with four;
    // 60000 x 720: 245 and 200.
    auto points = [&](int64_t blocks) { return div_up(a.n, groups < blocks ? blocks / groups : 1); };
    const int64_t few = points(2 * kCus), want = few > 512 ? points(4 * kCus) : few;
    a.chunk = want < 32 ? 32 : want > 4096 ? 4096 : div_up(want, 32) * 32;
    a.n_chunks = div_up(a.n, a.chunk);
    // Extents cost a fifth of the score: fewer chunks, so that a score block can
    // join them; a long cloud takes more and a launch that joins them.
    const int64_t per = div_up(a.n, kYawJoin), fill = div_up(a.n, div_up(2 * kCus, groups));
    a.ext_chunk = per < 64 ? 64 : per <= 2048 ? per : fill < 1024 ? 1024 : fill > 16384 ? 16384 : fill;
    a.n_ext = div_up(a.n, a.ext_chunk);
}

size_t yaw_doubles(const YawArgs& a)
{
    return (size_t)(a.K * a.n_chunks + (4 * (int64_t)a.K + 2) * (a.n_ext + 1) + 2 * (int64_t)a.K);
}

// The split's numbers of chunks rise and fall with the points and the yaws; this
// is at least yaw_doubles of any split of n points or fewer and K yaws or fewer.
// Score chunks hold 32 points at least, and there are at most 4 kCus / groups or
// one per 4096 points, of groups that hold at most 64 yaws each; extents chunks
// hold 64 points, and there are at most kYawJoin, or one per 1024 points and
// either 2 kCus / groups + 1 or one per 16384 points.
size_t yaw_doubles_most(int64_t n, int64_t K)
{
    const int64_t by_points = K * div_up(n, 32), by_blocks = 64 * 4 * kCus + K * div_up(n, 4096);
    const int64_t ext_points = K * div_up(n, 1024), ext_blocks = 64 * 2 * kCus + K + K * div_up(n, 16384);
    const int64_t sums = by_points < by_blocks ? by_points : by_blocks;
    const int64_t short_ext = div_up(n, 64) < kYawJoin ? div_up(n, 64) : kYawJoin;
    const int64_t ext = K * short_ext + (ext_points < ext_blocks ? ext_points : ext_blocks);
    const int64_t z = short_ext + div_up(n, 1024);
    return (size_t)(sums + 4 * (ext + K) + 2 * (z + 1) + 2 * K);
}

void yaw_place(YawArgs& a, double* ws)
{
    a.turn = (double2*)ws;
    a.part_sum = ws + 2 * (int64_t)a.K;
    a.part_ext = a.part_sum + a.K * a.n_chunks;
    a.part_z = a.part_ext + 4 * (int64_t)a.K * (a.n_ext + 1);
}

hipError_t launch_canonical_yaw(YawArgs a, hipStream_t s)
{
    const uint32_t groups = (uint32_t)div_up(a.K, 1 << a.log2_kl);
    hipError_t e;
    hipLaunchKernelGGL(k_yaw_extents, dim3((uint32_t)a.n_ext, groups), dim3(kYawThreads), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.n_ext > kYawJoin) {
        double* ext = a.part_ext + 4 * (int64_t)a.K * a.n_ext;
        double* z = a.part_z + 2 * a.n_ext;
        hipLaunchKernelGGL(k_yaw_join, dim3(1, groups), dim3(1024), 0, s, a, ext, z);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        a.part_ext = ext;
        a.part_z = z;
        a.n_ext = 1;
    }
    hipLaunchKernelGGL(k_yaw_score, dim3((uint32_t)a.n_chunks, groups), dim3(kYawThreads), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int log2_kf = 6;
    while (log2_kf > 0 && (1 << (log2_kf - 1)) >= a.K) --log2_kf;
    hipLaunchKernelGGL(k_yaw_finish, dim3(1), dim3(1024), 0, s, a, log2_kf);
    return hipGetLastError();
}

}  // namespace prenom
