// Reduced-precision form of the object-NeRF MLP: BF16 or FP16 operands on
// v_mfma_f32_16x16x16_{bf16,f16} with FP32 accumulation.  The FP32 master
// weights are converted once per block into LDS fragments; activations,
// deltas and every gradient stay FP32 in registers and are rounded only when
// they become an MFMA operand.
//
// Operand layouts of the 16x16x16 instruction (lane l, q = l/16, j = l%16):
// A[i][k] holds k = 4q..4q+3 of row i = j in lane l; B[k][n] holds
// k = 4q..4q+3 of column n = j; D[i][n] sits at lane n + 16*(i/4), register
// i%4.  So the four output registers of a 16-neuron tile are exactly the B
// operand of the next layer over that tile (k = 4q + r), with no permutation;
// weight fragments hold W[16 to + j][16 ti + 4q .. 4q+3].
//
// The weight gradient contracts over the 16 samples of a tile with one MFMA
// per (out tile, in tile), whose operands are staged in LDS in the MFMA type and
// read transposed; the 8 waves of a block merge their dW in LDS and write one
// partial.
#include "mlp_common.h"

namespace prenom {
namespace {

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

struct Bf16Op {
    using vec = short4_t;
    static __device__ __forceinline__ short cvt(float x) { return __builtin_bit_cast(short, (__bf16)x); }
    static __device__ __forceinline__ floatx4 mma(vec a, vec b, floatx4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
};

struct F16Op {
    using vec = half4_t;
    static __device__ __forceinline__ _Float16 cvt(float x) { return (_Float16)x; }
    static __device__ __forceinline__ floatx4 mma(vec a, vec b, floatx4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
    }
};

template <class P>
__device__ __forceinline__ typename P::vec pack(float a, float b, float c, float d)
{
    typename P::vec v;
    v[0] = P::cvt(a);
    v[1] = P::cvt(b);
    v[2] = P::cvt(c);
    v[3] = P::cvt(d);
    return v;
}

template <class P>
__device__ __forceinline__ typename P::vec pack(floatx4 x)
{
    return pack<P>(x[0], x[1], x[2], x[3]);
}

// ReLU decisions of one sample and lane group q as bits: bit 4 to + r for neuron
// 16 to + 4 q + r (the decision of the FP32 pre-activation, whatever the 16-bit
// activation rounds to).
template <int OT>
__device__ __forceinline__ uint32_t relu_mask_bits(const floatx4 (&h)[OT])
{
    static_assert(4 * OT <= 32, "mask bits per lane");
    uint32_t m = 0;
#pragma unroll
    for (int to = 0; to < OT; ++to)
#pragma unroll
        for (int r = 0; r < 4; ++r) m |= (h[to][r] > 0.0f ? 1u : 0u) << (4 * to + r);
    return m;
}

__device__ __forceinline__ floatx4 mask_by_bits(floatx4 g, uint32_t m, int to)
{
    return {(m >> (4 * to)) & 1u ? g[0] : 0.0f, (m >> (4 * to + 1)) & 1u ? g[1] : 0.0f,
            (m >> (4 * to + 2)) & 1u ? g[2] : 0.0f, (m >> (4 * to + 3)) & 1u ? g[3] : 0.0f};
}

template <int IN, int W, int D>
struct NetLp {
    static constexpr int KB1 = (IN + 15) / 16;  // 16-feature K-blocks of layer 1 (zero-padded)
    static constexpr int OT = W / 16;         // 16-neuron tiles of a hidden layer
    static constexpr int IT = (IN + 15) / 16; // 16-feature tiles of the input
    static constexpr int F1 = 0;                        // [OT][KB1]
    static constexpr int FH = F1 + OT * KB1;            // [D-1][OT][OT]
    static constexpr int FO = FH + (D - 1) * OT * OT;   // [OT]
    static constexpr int N_FWD = FO + OT;
    static constexpr int BO = N_FWD;                    // [OT]
    static constexpr int BH = BO + OT;                  // [D-1][OT][OT]
    static constexpr int B1 = BH + (D - 1) * OT * OT;   // [IT][OT]
    static constexpr int N_ALL = B1 + IT * OT;
    static constexpr int OFF_W1 = 0;
    static constexpr int OFF_H = W * IN;
    static constexpr int OFF_OUT = W * IN + (D - 1) * W * W;
    static constexpr int N_PARAMS = OFF_OUT + 4 * W;
    static_assert(IN % 8 == 0 && W % 16 == 0 && D >= 1, "shape");
};

// Weight fragments: fragment f, lane l holds 4 consecutive K values.
template <int IN, int W, int D, class P>
__device__ __forceinline__ void load_fragments_lp(const float* __restrict__ w, typename P::vec* __restrict__ frag, int n_frag, int f0 = 0)
{
    using N = NetLp<IN, W, D>;
    for (int idx = threadIdx.x; idx < n_frag * 64; idx += blockDim.x) {
        const int f = f0 + (idx >> 6), l = idx & 63, q = l >> 4, j = l & 15;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float x;
            if (f < N::FH) {  // W1[16 to + j][16 m + 4 q + r], features >= IN zero
                const int to = f / N::KB1, m = f % N::KB1, col = 16 * m + 4 * q + r;
                x = col < IN ? w[N::OFF_W1 + (16 * to + j) * IN + col] : 0.0f;
            } else if (f < N::FO) {  // Wk[16 to + j][16 ti + 4 q + r]
                const int g = f - N::FH, k = g / (N::OT * N::OT), rem = g % (N::OT * N::OT);
                const int to = rem / N::OT, ti = rem % N::OT;
                x = w[N::OFF_H + k * W * W + (16 * to + j) * W + 16 * ti + 4 * q + r];
            } else if (f < N::N_FWD) {  // Wout[j][16 ti + 4 q + r], rows >= 4 zero
                const int ti = f - N::FO;
                x = j < 4 ? w[N::OFF_OUT + j * W + 16 * ti + 4 * q + r] : 0.0f;
            } else if (f < N::BH) {  // Wout^T over the 4 outputs: k = 4 q + r < 4
                const int to = f - N::BO;
                x = q == 0 ? w[N::OFF_OUT + r * W + 16 * to + j] : 0.0f;
            } else if (f < N::B1) {  // Wk^T: Wk[16 ti + 4 q + r][16 to + j]
                const int g = f - N::BH, k = g / (N::OT * N::OT), rem = g % (N::OT * N::OT);
                const int to = rem / N::OT, ti = rem % N::OT;
                x = w[N::OFF_H + k * W * W + (16 * ti + 4 * q + r) * W + 16 * to + j];
            } else {  // W1^T: W1[16 ti + 4 q + r][16 to + j], columns >= IN zero
                const int g = f - N::B1, to = g / N::OT, ti = g % N::OT, col = 16 * to + j;
                x = col < IN ? w[N::OFF_W1 + (16 * ti + 4 * q + r) * IN + col] : 0.0f;
            }
            v[r] = x;
        }
        frag[idx] = pack<P>(v[0], v[1], v[2], v[3]);
    }
}

// Layer-1 inputs of one lane: features 16 m + 4 q + r of sample s (levels
// 8 m + 2 q and 8 m + 2 q + 1 of the level-major feature array); features
// beyond IN are zero.
template <int IN, int KB1>
__device__ __forceinline__ void load_inputs_lp(const float2* __restrict__ y, int64_t n_s, int64_t s, bool valid, int q,
                                               floatx4 (&yf)[KB1])
{
#pragma unroll
    for (int m = 0; m < KB1; ++m) {
        float2 a = make_float2(0.0f, 0.0f), b = make_float2(0.0f, 0.0f);
        const int l0 = 8 * m + 2 * q;
        if (valid && 2 * l0 < IN) a = y[(int64_t)l0 * n_s + s];
        if (valid && 2 * (l0 + 1) < IN) b = y[(int64_t)(l0 + 1) * n_s + s];
        yf[m] = {a.x, a.y, b.x, b.y};
    }
}

// acc[to] = sum_ti A(fragment f0 + to * stride + ti) x b[ti], K-blocks outer
// and output tiles inner (independent accumulators interleave), with a
// scheduling fence every kFence K-blocks so fragment loads are not all hoisted.
template <class P, int OT, int KT, int kFence = 4>
__device__ __forceinline__ void layer_lp_ks_outer(const typename P::vec* __restrict__ frag, int lane, int f0, int stride,
                                                  const typename P::vec (&b)[KT], floatx4 (&acc)[OT])
{
#pragma unroll
    for (int to = 0; to < OT; ++to) acc[to] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ti = 0; ti < KT; ++ti) {
#pragma unroll
        for (int to = 0; to < OT; ++to) acc[to] = P::mma(frag[(f0 + to * stride + ti) * 64 + lane], b[ti], acc[to]);
        if (ti % kFence == kFence - 1) __builtin_amdgcn_sched_barrier(0);
    }
}

template <int IN, int W, int D, class P>
__device__ __forceinline__ void chain_lp(const typename P::vec* __restrict__ frag, int lane,
                                         const floatx4 (&yf)[NetLp<IN, W, D>::KB1],
                                         floatx4 (&hs)[D][NetLp<IN, W, D>::OT], floatx4& o)
{
    using N = NetLp<IN, W, D>;
    if constexpr (W >= kWideWidth) {
        typename P::vec b1[N::KB1];
#pragma unroll
        for (int m = 0; m < N::KB1; ++m) b1[m] = pack<P>(yf[m]);
        floatx4 acc[N::OT];
        layer_lp_ks_outer<P, N::OT, N::KB1>(frag, lane, N::F1, N::KB1, b1, acc);
#pragma unroll
        for (int to = 0; to < N::OT; ++to) hs[0][to] = relu4(acc[to]);
#pragma unroll
        for (int k = 1; k < D; ++k) {
            typename P::vec b[N::OT];
#pragma unroll
            for (int ti = 0; ti < N::OT; ++ti) b[ti] = pack<P>(hs[k - 1][ti]);
            layer_lp_ks_outer<P, N::OT, N::OT>(frag, lane, N::FH + (k - 1) * N::OT * N::OT, N::OT, b, acc);
#pragma unroll
            for (int to = 0; to < N::OT; ++to) hs[k][to] = relu4(acc[to]);
        }
    } else {
#pragma unroll
        for (int to = 0; to < N::OT; ++to) {
            floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int m = 0; m < N::KB1; ++m) acc = P::mma(frag[(N::F1 + to * N::KB1 + m) * 64 + lane], pack<P>(yf[m]), acc);
            hs[0][to] = relu4(acc);
        }
#pragma unroll
        for (int k = 1; k < D; ++k) {
#pragma unroll
            for (int to = 0; to < N::OT; ++to) {
                floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ti = 0; ti < N::OT; ++ti)
                    acc = P::mma(frag[(N::FH + ((k - 1) * N::OT + to) * N::OT + ti) * 64 + lane], pack<P>(hs[k - 1][ti]), acc);
                hs[k][to] = relu4(acc);
            }
        }
    }
    o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ti = 0; ti < N::OT; ++ti) o = P::mma(frag[(N::FO + ti) * 64 + lane], pack<P>(hs[D - 1][ti]), o);
}

template <int IN, int W, int D, class P>
__device__ __forceinline__ void mlp_fwd_tiles_lp(const typename P::vec* __restrict__ frag,
                                                 const float2* __restrict__ y, int64_t n_s, float4* __restrict__ sc,
                                                 int64_t tile0, int64_t end, int64_t step)
{
    using N = NetLp<IN, W, D>;
    const int lane = threadIdx.x & 63, q = lane >> 4, j = lane & 15;
    floatx4 yn[N::KB1];  // the next tile's inputs, loaded while the current tile runs
    if (tile0 < end) load_inputs_lp<IN, N::KB1>(y, n_s, tile0 * 16 + j, tile0 * 16 + j < n_s, q, yn);
    for (int64_t tile = tile0; tile < end; tile += step) {
        const int64_t s = tile * 16 + j;
        const bool valid = s < n_s;
        floatx4 yf[N::KB1];
#pragma unroll
        for (int m = 0; m < N::KB1; ++m) yf[m] = yn[m];
        const int64_t sn = (tile + step) * 16 + j;
        if (tile + step < end) load_inputs_lp<IN, N::KB1>(y, n_s, sn, sn < n_s, q, yn);
        floatx4 hs[D][N::OT];
        floatx4 o;
        chain_lp<IN, W, D, P>(frag, lane, yf, hs, o);
        if (q == 0 && valid) sc[s] = make_float4(__expf(o[0]), sigmoidf_(o[1]), sigmoidf_(o[2]), sigmoidf_(o[3]));
    }
}

// Three waves per SIMD: without the hint the 128-wide shapes take 136 VGPRs and 32
// AGPRs, with it at most 114; the forward of 48 objects 3.09 -> 2.96 ms.
template <int IN, int W, int D, class P>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_fwd_lp(
    const float* __restrict__ w, const float2* __restrict__ y, int64_t n_s, float4* __restrict__ sc)
{
    using N = NetLp<IN, W, D>;
    extern __shared__ __align__(16) unsigned char smem_f[];
    typename P::vec* frag = reinterpret_cast<typename P::vec*>(smem_f);
    load_fragments_lp<IN, W, D, P>(w, frag, N::N_FWD);
    __syncthreads();
    const int64_t wave0 = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int64_t n_waves = (int64_t)gridDim.x * (blockDim.x / 64);
    mlp_fwd_tiles_lp<IN, W, D, P>(frag, y, n_s, sc, wave0, (n_s + 15) / 16, n_waves);
}

template <int IN, int W, int D, class P>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_fwd_lp_batch(
    const MlpWork* __restrict__ work, const float* __restrict__ params, const float2* __restrict__ y,
    float4* __restrict__ sc)
{
    using N = NetLp<IN, W, D>;
    extern __shared__ __align__(16) unsigned char smem_f[];
    typename P::vec* frag = reinterpret_cast<typename P::vec*>(smem_f);
    const MlpWork wk = work[blockIdx.x];
    load_fragments_lp<IN, W, D, P>(params + wk.w_off, frag, N::N_FWD);
    __syncthreads();
    mlp_fwd_tiles_lp<IN, W, D, P>(frag, y + wk.y_off / 2, wk.n_s, sc + wk.s_off,
                                  wk.tile_begin + (threadIdx.x >> 6), wk.tile_end, blockDim.x / 64);
}

// The weight gradient contracts over samples, so its operands hold four samples
// of a neuron, where the tiles hold four neurons of a sample.  The arrays are
// staged in LDS in the MFMA type, a row per sample, and read transposed: a lane
// writes its four neurons in 8 bytes, and ds_read_b64_tr_b16 hands lane (q, j) of
// a 16-lane group neuron j of the four rows whose 8-byte pieces the group's
// lanes address (lane 4 r + c: row r, piece c).  Rows are 8 banks apart modulo
// the 64 banks, so that the reads of 8 rows meet no bank twice.
constexpr int lds_pitch(int halves)  // of a staged row, in halfwords: 16 modulo 32
{
    return (halves + 31) / 32 * 32 + 16;
}

template <class V>
__device__ __forceinline__ V read_transposed(const uint16_t* p)
{
    return __builtin_bit_cast(
        V, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t*)p));
}

template <class V>
__device__ __forceinline__ void write_staged(uint16_t* p, V v)
{
    *reinterpret_cast<uint2*>(p) = __builtin_bit_cast(uint2, v);
}

template <int IN, int W, int D>
struct BwdLdsLp {
    static constexpr int IP = 16 * NetLp<IN, W, D>::IT;
    static constexpr int PITCH = lds_pitch(W > IP ? W : IP);
    static constexpr int PER_WAVE = 16 * PITCH;  // floats: two staged arrays of 16 rows of halfwords
};

// dw += delta h^T over the wave's 16 staged samples; dp and hp are where the
// lane's transposed reads begin.
template <int OTILES, int ITILES, class P>
__device__ __forceinline__ void accumulate_dw_lp(const uint16_t* __restrict__ dp, const uint16_t* __restrict__ hp,
                                                 floatx4 (&dw)[OTILES][ITILES])
{
    typename P::vec a[OTILES], b[ITILES];
#pragma unroll
    for (int to = 0; to < OTILES; ++to) a[to] = read_transposed<typename P::vec>(dp + 16 * to);
#pragma unroll
    for (int ti = 0; ti < ITILES; ++ti) b[ti] = read_transposed<typename P::vec>(hp + 16 * ti);
#pragma unroll
    for (int to = 0; to < OTILES; ++to)
#pragma unroll
        for (int ti = 0; ti < ITILES; ++ti) dw[to][ti] = P::mma(a[to], b[ti], dw[to][ti]);
}

// Backward over tiles tile0, tile0 + step, ... < end of one object whose
// fragments are at the start of smem_lp; called by every thread of the block.
template <int IN, int W, int D, class P>
__device__ __forceinline__ void mlp_bwd_tiles_lp(unsigned char* __restrict__ smem_lp, const float2* __restrict__ y,
                                 const float4* __restrict__ dout, int64_t n_s, float2* __restrict__ dy,
                                 float* __restrict__ dst, int64_t tile0, int64_t end, int64_t step)
{
    using N = NetLp<IN, W, D>;
    using B = BwdLdsLp<IN, W, D>;
    const typename P::vec* frag = reinterpret_cast<const typename P::vec*>(smem_lp);
    float* stage = reinterpret_cast<float*>(smem_lp + sizeof(typename P::vec) * N::N_ALL * 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4, j = lane & 15;
    uint16_t* sD = reinterpret_cast<uint16_t*>(stage + wave * B::PER_WAVE);
    uint16_t* sH = sD + 16 * B::PITCH;
    const int wr = j * B::PITCH + 4 * q, rd = (4 * q + j / 4) * B::PITCH + 4 * (j & 3);  // the lane's writes and reads

    floatx4 dW1[N::OT][N::IT];
    floatx4 dWh[D > 1 ? D - 1 : 1][N::OT][N::OT];
    floatx4 dWo[1][N::OT];
#pragma unroll
    for (int a = 0; a < N::OT; ++a) {
#pragma unroll
        for (int b = 0; b < N::IT; ++b) dW1[a][b] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int b = 0; b < N::OT; ++b)
#pragma unroll
            for (int k = 0; k < (D > 1 ? D - 1 : 1); ++k) dWh[k][a][b] = {0.0f, 0.0f, 0.0f, 0.0f};
        dWo[0][a] = {0.0f, 0.0f, 0.0f, 0.0f};
    }

    // the next tile's inputs and upstream gradient, loaded while the current tile runs
    floatx4 yn[N::KB1];
    float4 gn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    auto load_tile = [&](int64_t t) {
        const int64_t st = t * 16 + j;
        const bool ok = t < end && st < n_s;
        load_inputs_lp<IN, N::KB1>(y, n_s, st, ok, q, yn);
        gn = ok && q == 0 ? dout[st] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    };
    load_tile(tile0);
    for (int64_t tile = tile0; tile < end; tile += step) {
        const int64_t s = tile * 16 + j;
        const bool valid = s < n_s;
        floatx4 yf[N::KB1];
#pragma unroll
        for (int m = 0; m < N::KB1; ++m) yf[m] = yn[m];
        const float4 gc = gn;
        load_tile(tile + step);
        floatx4 hs[D][N::OT];
        floatx4 o;
        chain_lp<IN, W, D, P>(frag, lane, yf, hs, o);

        // head adjoint in the output tile's own layout (rows 4q + r; only q == 0 is real)
        floatx4 dO[1] = {{0.0f, 0.0f, 0.0f, 0.0f}};
        if (q == 0 && valid) {
            const float4 g = gc;
            const float c1 = sigmoidf_(o[1]), c2 = sigmoidf_(o[2]), c3 = sigmoidf_(o[3]);
            dO[0] = {g.x * __expf(o[0]), g.y * c1 * (1.0f - c1), g.z * c2 * (1.0f - c2), g.w * c3 * (1.0f - c3)};
        }
        const typename P::vec dOp = pack<P>(dO[0]);
        wave_lds_sync();
        write_staged(sD + wr, dOp);
#pragma unroll
        for (int ti = 0; ti < N::OT; ++ti) write_staged(sH + wr + 16 * ti, pack<P>(hs[D - 1][ti]));
        wave_lds_sync();
        accumulate_dw_lp<1, N::OT, P>(sD + rd, sH + rd, dWo);

        floatx4 delta[N::OT];
#pragma unroll
        for (int to = 0; to < N::OT; ++to) {
            floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
            acc = P::mma(frag[(N::BO + to) * 64 + lane], dOp, acc);
            delta[to] = mask_pos(acc, hs[D - 1][to]);
        }
#pragma unroll
        for (int k = D - 1; k >= 1; --k) {
            typename P::vec dp[N::OT];
#pragma unroll
            for (int ti = 0; ti < N::OT; ++ti) dp[ti] = pack<P>(delta[ti]);
            wave_lds_sync();
#pragma unroll
            for (int ti = 0; ti < N::OT; ++ti) {
                write_staged(sD + wr + 16 * ti, dp[ti]);
                write_staged(sH + wr + 16 * ti, pack<P>(hs[k - 1][ti]));
            }
            wave_lds_sync();
            accumulate_dw_lp<N::OT, N::OT, P>(sD + rd, sH + rd, dWh[k - 1]);
#pragma unroll
            for (int to = 0; to < N::OT; ++to) {
                floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ti = 0; ti < N::OT; ++ti)
                    acc = P::mma(frag[(N::BH + ((k - 1) * N::OT + to) * N::OT + ti) * 64 + lane], dp[ti], acc);
                delta[to] = mask_pos(acc, hs[k - 1][to]);
            }
        }
        // layer 1: stage delta and the inputs (features 16 m + 4 q + r of sample j, zero beyond IN)
        typename P::vec dp[N::OT];
#pragma unroll
        for (int ti = 0; ti < N::OT; ++ti) dp[ti] = pack<P>(delta[ti]);
        wave_lds_sync();
#pragma unroll
        for (int ti = 0; ti < N::OT; ++ti) write_staged(sD + wr + 16 * ti, dp[ti]);
#pragma unroll
        for (int m = 0; m < N::KB1; ++m) write_staged(sH + wr + 16 * m, pack<P>(yf[m]));
        wave_lds_sync();
        accumulate_dw_lp<N::OT, N::IT, P>(sD + rd, sH + rd, dW1);
#pragma unroll
        for (int to = 0; to < N::IT; ++to) {
            floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ti = 0; ti < N::OT; ++ti) acc = P::mma(frag[(N::B1 + to * N::OT + ti) * 64 + lane], dp[ti], acc);
            const int f = 16 * to + 4 * q;  // features f..f+3 = levels f/2 and f/2 + 1
            if (valid && f < IN) {
                dy[(int64_t)(f >> 1) * n_s + s] = make_float2(acc[0], acc[1]);
                dy[(int64_t)((f >> 1) + 1) * n_s + s] = make_float2(acc[2], acc[3]);
            }
        }
    }

    static_assert(N::N_PARAMS <= kBwdWaves * B::PER_WAVE, "reduction buffer");
    float* red = stage;
    __syncthreads();
    for (int wv = 0; wv < kBwdWaves; ++wv) {
        if (wave == wv) {
            merge_dw<N::OT, N::IT>(red + N::OFF_W1, dW1, W, IN, q, j, wv == 0);
#pragma unroll
            for (int k = 1; k < D; ++k)
                merge_dw<N::OT, N::OT>(red + N::OFF_H + (k - 1) * W * W, dWh[k - 1], W, W, q, j, wv == 0);
            merge_dw<1, N::OT>(red + N::OFF_OUT, dWo, 4, W, q, j, wv == 0);
        }
        __syncthreads();
    }
    for (int p = threadIdx.x; p < N::N_PARAMS; p += blockDim.x) dst[p] = red[p];
}

template <int IN, int W, int D, class P>
__global__ __launch_bounds__(64 * kBwdWaves) void k_mlp_bwd_lp(const float* __restrict__ w,
                                                               const float2* __restrict__ y,
                                                               const float4* __restrict__ dout, int64_t n_s,
                                                               float2* __restrict__ dy, float* __restrict__ partial)
{
    using N = NetLp<IN, W, D>;
    extern __shared__ __align__(16) unsigned char smem_lp[];
    load_fragments_lp<IN, W, D, P>(w, reinterpret_cast<typename P::vec*>(smem_lp), N::N_ALL);
    __syncthreads();
    const int64_t wave0 = (int64_t)blockIdx.x * kBwdWaves + (threadIdx.x >> 6);
    mlp_bwd_tiles_lp<IN, W, D, P>(smem_lp, y, dout, n_s, dy, partial + (int64_t)blockIdx.x * N::N_PARAMS, wave0,
                                  (n_s + 15) / 16, (int64_t)gridDim.x * kBwdWaves);
}

template <int IN, int W, int D, class P>
__global__ __launch_bounds__(64 * kBwdWaves) void k_mlp_bwd_lp_batch(const MlpWork* __restrict__ work,
                                                                     const float* __restrict__ params,
                                                                     const float2* __restrict__ y,
                                                                     const float4* __restrict__ dout,
                                                                     float2* __restrict__ dy,
                                                                     float* __restrict__ partial, int64_t slot_stride)
{
    using N = NetLp<IN, W, D>;
    extern __shared__ __align__(16) unsigned char smem_lp[];
    const MlpWork wk = work[blockIdx.x];
    load_fragments_lp<IN, W, D, P>(params + wk.w_off, reinterpret_cast<typename P::vec*>(smem_lp), N::N_ALL);
    __syncthreads();
    mlp_bwd_tiles_lp<IN, W, D, P>(smem_lp, y + wk.y_off / 2, dout + wk.s_off, wk.n_s, dy + wk.y_off / 2,
                                  partial + (int64_t)blockIdx.x * slot_stride, wk.tile_begin + (threadIdx.x >> 6),
                                  wk.tile_end, kBwdWaves);
}

// ---------------------------------------------------------------- 128 wide
// The 128-wide backward is one kernel: a block takes its samples 128 at a time,
// one 16-sample tile per wave, recomputes the forward, runs the transposed chain
// and accumulates the weight gradient, whose operands (four consecutive samples
// of a neuron) go through LDS: deltas and activations of the 128 samples in the
// MFMA type.  The waves split the output rows, 16 each, so the
// block's partial is written without a merge.  Forward and transposed fragments
// (86 KB with two layers) and the two staged arrays (72 KB) fill a CU's LDS.
// Nothing but the features, the head outputs and their adjoint is read: storing
// the activations in the forward and the deltas between a chain and a
// weight-gradient kernel moved 2.5 KB a sample and ran at the HBM's rate (48
// objects, 28.5 M samples 128 wide: forward 4.0 and backward 10.3 ms).
constexpr int kWideWavesLp = 8;
constexpr int kWideChunk = 16 * kWideWavesLp;  // samples staged at a time
constexpr int kHeadPitch = kWideChunk + 8;     // halfwords per row of the staged head adjoint

template <int IN, int W, int D>
struct WideLdsLp {
    using N = NetLp<IN, W, D>;
    static constexpr int N_FRAG = N::FO + (N::N_ALL - N::N_FWD);  // hidden forward fragments, then the transposed ones
    // staged arrays, a row per sample, in halfwords from the end of the fragments
    static constexpr int PITCH = lds_pitch(W);
    static constexpr int A = 0;
    static constexpr int B = A + kWideChunk * PITCH;
    static constexpr int Y_PITCH = D == 1 ? lds_pitch(16 * N::IT) : PITCH;
    static constexpr int Y = D == 1 ? B + kWideChunk * PITCH : B;  // inputs: beside the others, or in place of B
    static constexpr int DO = D == 1 ? Y + kWideChunk * Y_PITCH : B + kWideChunk * PITCH;  // head adjoint: 4 rows of samples
    static constexpr int HALVES = DO + 4 * kHeadPitch;
    static constexpr size_t BYTES = (size_t)N_FRAG * 512 + sizeof(uint16_t) * (size_t)HALVES;
    static_assert(BYTES <= 160 * 1024 && (IN <= 32 && D <= 2), "LDS of one CU");
};

// Tiles [tile0, tile1) of one object: dy of their samples and their share of
// the weight gradient to dst.  Called by every thread of the block.
template <int IN, int W, int D, class P>
__device__ __forceinline__ void mlp_wide_bwd_lp(unsigned char* __restrict__ smem, const float* __restrict__ w,
                                                const float2* __restrict__ y, const float4* __restrict__ sc,
                                                const float4* __restrict__ dout, int64_t n_s, float2* __restrict__ dy,
                                                float* __restrict__ dst, int64_t tile0, int64_t tile1)
{
    using N = NetLp<IN, W, D>;
    using L = WideLdsLp<IN, W, D>;
    using vec = typename P::vec;
    constexpr int kFence = 2;  // (four would spill)
    static_assert(N::OT == kWideWavesLp, "one row tile per wave");
    vec* ffrag = reinterpret_cast<vec*>(smem);
    vec* bfrag = ffrag + N::FO * 64;
    uint16_t* st = reinterpret_cast<uint16_t*>(smem + (size_t)L::N_FRAG * 512);
    constexpr int BO = 0, BH = N::BH - N::N_FWD, B1 = N::B1 - N::N_FWD;  // rebased to bfrag
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4, j = lane & 15;
    load_fragments_lp<IN, W, D, P>(w, ffrag, N::FO);
    load_fragments_lp<IN, W, D, P>(w, bfrag, N::N_ALL - N::N_FWD, N::N_FWD);
    const int col = 16 * wave + j;  // the lane's sample within the chunk
    // neurons 16 t + 4 q .. + 3 of sample `col`, into a staged array
    auto put = [&](int base, int pitch, int t, vec v) { write_staged(st + base + col * pitch + 16 * t + 4 * q, v); };
    // samples 16 ks + 4 q .. + 3 of neuron 16 t + j: an MFMA operand
    const int row = 4 * q + j / 4, piece = 4 * (j & 3);
    auto op = [&](int base, int pitch, int t, int ks) {
        return read_transposed<vec>(st + base + (16 * ks + row) * pitch + 16 * t + piece);
    };
    floatx4 aH[N::OT], a1[N::IT], aO = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < N::OT; ++t) aH[t] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < N::IT; ++t) a1[t] = {0.0f, 0.0f, 0.0f, 0.0f};
    // W_out: A[i][k] = dO_i (rows i >= 4 zero), B = the last layer's activations
    auto add_out = [&](int hbase) {
#pragma unroll 2
        for (int ks = 0; ks < kWideChunk / 16; ++ks) {
            vec d = __builtin_bit_cast(
                vec, *reinterpret_cast<const uint2*>(st + L::DO + (j & 3) * kHeadPitch + 16 * ks + 4 * q));
            if (j >= 4) d = pack<P>(0.0f, 0.0f, 0.0f, 0.0f);
            aO = P::mma(d, op(hbase, L::PITCH, wave, ks), aO);
        }
    };
    auto add_in = [&](int dbase) {  // W_1
#pragma unroll 2
        for (int ks = 0; ks < kWideChunk / 16; ++ks) {
            const vec av = op(dbase, L::PITCH, wave, ks);
#pragma unroll
            for (int t = 0; t < N::IT; ++t) a1[t] = P::mma(av, op(L::Y, L::Y_PITCH, t, ks), a1[t]);
        }
    };
    // the next tile's inputs, upstream gradient and head outputs, loaded while
    // the current tile runs (lanes q == 0 hold the head's four outputs)
    floatx4 yn[N::KB1];
    float4 gn, vn;
    auto load_tile = [&](int64_t t) {
        const int64_t s = t * 16 + j;
        const bool ok = t < tile1 && s < n_s;
        load_inputs_lp<IN, N::KB1>(y, n_s, s, ok, q, yn);
        gn = vn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (ok && q == 0) {
            gn = dout[s];
            vn = sc[s];
        }
    };
    load_tile(tile0 + wave);
    __syncthreads();
    for (int64_t c0 = tile0; c0 < tile1; c0 += kWideWavesLp) {
        const int64_t tile = c0 + wave, s = tile * 16 + j;
        const bool valid = tile < tile1 && s < n_s;
        vec yp[N::KB1], hp[D][N::OT];
        uint32_t mask[D];
#pragma unroll
        for (int m = 0; m < N::KB1; ++m) yp[m] = pack<P>(yn[m]);
        const float4 g = gn, v = vn;
        load_tile(tile + kWideWavesLp);
        floatx4 acc[N::OT];
        layer_lp_ks_outer<P, N::OT, N::KB1>(ffrag, lane, N::F1, N::KB1, yp, acc);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (k > 0)
                layer_lp_ks_outer<P, N::OT, N::OT, kFence>(ffrag, lane, N::FH + (k - 1) * N::OT * N::OT, N::OT, hp[k > 0 ? k - 1 : 0],
                                                   acc);
#pragma unroll
            for (int to = 0; to < N::OT; ++to) acc[to] = relu4(acc[to]);
            mask[k] = relu_mask_bits(acc);
#pragma unroll
            for (int to = 0; to < N::OT; ++to) hp[k][to] = pack<P>(acc[to]);
        }
        // head adjoint: d sigma / d o0 = sigma, d c / d o = c (1 - c)
        const vec dO = pack<P>(g.x * v.x, g.y * v.y * (1.0f - v.y), g.z * v.z * (1.0f - v.z), g.w * v.w * (1.0f - v.w));
        vec dp[N::OT];
#pragma unroll
        for (int to = 0; to < N::OT; ++to) {
            const floatx4 d = P::mma(bfrag[(BO + to) * 64 + lane], dO, floatx4{0.0f, 0.0f, 0.0f, 0.0f});
            dp[to] = pack<P>(mask_by_bits(d, mask[D - 1], to));
        }
        auto put_out = [&] {
            if (q == 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const auto x = dO[r];
                    st[L::DO + r * kHeadPitch + col] = __builtin_bit_cast(uint16_t, x);
                }
            }
        };
        auto store_dy = [&] {
            floatx4 gy[N::IT];
            layer_lp_ks_outer<P, N::IT, N::OT, kFence>(bfrag, lane, B1, N::OT, dp, gy);
#pragma unroll
            for (int to = 0; to < N::IT; ++to) {
                const int f = 16 * to + 4 * q;
                if (valid && f < IN) {
                    dy[(int64_t)(f >> 1) * n_s + s] = make_float2(gy[to][0], gy[to][1]);
                    dy[(int64_t)((f >> 1) + 1) * n_s + s] = make_float2(gy[to][2], gy[to][3]);
                }
            }
        };
        __syncthreads();  // the previous chunk's operands have been read
        if constexpr (D == 1) {
#pragma unroll
            for (int to = 0; to < N::OT; ++to) {
                put(L::A, L::PITCH, to, dp[to]);
                put(L::B, L::PITCH, to, hp[0][to]);
            }
#pragma unroll
            for (int m = 0; m < N::KB1; ++m) put(L::Y, L::Y_PITCH, m, yp[m]);
            put_out();
            __syncthreads();
            add_out(L::B);
            store_dy();
            add_in(L::A);
        } else {
            // the last activations in A until W_out's gradient has them, then the deltas
#pragma unroll
            for (int to = 0; to < N::OT; ++to) {
                put(L::A, L::PITCH, to, hp[D - 1][to]);
                put(L::B, L::PITCH, to, hp[0][to]);
            }
            put_out();
            __syncthreads();
            add_out(L::A);
            layer_lp_ks_outer<P, N::OT, N::OT, kFence>(bfrag, lane, BH, N::OT, dp, acc);
            __syncthreads();
#pragma unroll
            for (int to = 0; to < N::OT; ++to) {
                put(L::A, L::PITCH, to, dp[to]);
                dp[to] = pack<P>(mask_by_bits(acc[to], mask[0], to));
            }
            __syncthreads();
#pragma unroll 2
            for (int ks = 0; ks < kWideChunk / 16; ++ks) {
                const vec av = op(L::A, L::PITCH, wave, ks);
#pragma unroll
                for (int t = 0; t < N::OT; ++t) aH[t] = P::mma(av, op(L::B, L::PITCH, t, ks), aH[t]);
            }
            store_dy();
            __syncthreads();
#pragma unroll
            for (int to = 0; to < N::OT; ++to) put(L::A, L::PITCH, to, dp[to]);
#pragma unroll
            for (int m = 0; m < N::KB1; ++m) put(L::Y, L::Y_PITCH, m, yp[m]);
            __syncthreads();
            add_in(L::A);
        }
    }
    // D layout: row 16 wave + 4 q + r, column 16 t + j
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * wave + 4 * q + r;
#pragma unroll
        for (int t = 0; t < N::IT; ++t)
            if (16 * t + j < IN) dst[N::OFF_W1 + row * IN + 16 * t + j] = a1[t][r];
        if constexpr (D > 1) {
#pragma unroll
            for (int t = 0; t < N::OT; ++t) dst[N::OFF_H + row * W + 16 * t + j] = aH[t][r];
        }
        if (q == 0) dst[N::OFF_OUT + r * W + 16 * wave + j] = aO[r];
    }
}

template <int IN, int W, int D, class P>
__global__ __launch_bounds__(64 * kWideWavesLp) void k_mlp_wide_bwd_lp(const float* __restrict__ w,
                                                                       const float2* __restrict__ y,
                                                                       const float4* __restrict__ sc,
                                                                       const float4* __restrict__ dout, int64_t n_s,
                                                                       int64_t tiles_per_block,
                                                                       float2* __restrict__ dy,
                                                                       float* __restrict__ partial)
{
    extern __shared__ __align__(16) unsigned char smem_w[];
    const int64_t n_t = (n_s + 15) / 16, t0 = min((int64_t)blockIdx.x * tiles_per_block, n_t);
    mlp_wide_bwd_lp<IN, W, D, P>(smem_w, w, y, sc, dout, n_s, dy, partial + (int64_t)blockIdx.x * NetLp<IN, W, D>::N_PARAMS,
                                 t0, min(t0 + tiles_per_block, n_t));
}

template <int IN, int W, int D, class P>
__global__ __launch_bounds__(64 * kWideWavesLp) void k_mlp_wide_bwd_lp_batch(const MlpWork* __restrict__ work,
                                                                             const float* __restrict__ params,
                                                                             const float* __restrict__ y,
                                                                             const float4* __restrict__ sc,
                                                                             const float4* __restrict__ dout,
                                                                             float2* __restrict__ dy,
                                                                             float* __restrict__ partial,
                                                                             int64_t slot_stride)
{
    extern __shared__ __align__(16) unsigned char smem_w[];
    const MlpWork wk = work[blockIdx.x];
    mlp_wide_bwd_lp<IN, W, D, P>(smem_w, params + wk.w_off, reinterpret_cast<const float2*>(y + wk.y_off), sc + wk.s_off,
                                 dout + wk.s_off, wk.n_s, dy + wk.y_off / 2, partial + (int64_t)blockIdx.x * slot_stride,
                                 wk.tile_begin, wk.tile_end);
}

template <class K>
hipError_t set_lds_lp(K kern, size_t bytes)
{
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int IN, int W, int D, class P>
size_t fwd_lds_lp()
{
    return sizeof(typename P::vec) * (size_t)NetLp<IN, W, D>::N_FWD * 64;
}

template <int IN, int W, int D, class P>
size_t bwd_lds_lp()
{
    return sizeof(typename P::vec) * (size_t)NetLp<IN, W, D>::N_ALL * 64 +
           sizeof(float) * (size_t)kBwdWaves * BwdLdsLp<IN, W, D>::PER_WAVE;
}

template <int IN, int W, int D, class P>
hipError_t fwd_lp(const float* w, const float* y, int64_t n_s, float* sc, hipStream_t s)
{
    const int64_t n_tiles = (n_s + 15) / 16;
    const size_t lds = fwd_lds_lp<IN, W, D, P>();
    const int64_t blocks = fwd_blocks(n_tiles, 4, lds);
    hipError_t e = set_lds_lp(k_mlp_fwd_lp<IN, W, D, P>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_mlp_fwd_lp<IN, W, D, P>), dim3((uint32_t)blocks), dim3(256), lds, s, w, (const float2*)y,
                       n_s, (float4*)sc);
    return hipGetLastError();
}

template <int IN, int W, int D, class P>
hipError_t bwd_lp(const float* w, const float* y, const float* dout, const float* sc, int64_t n_s, float* dy,
                  float* partial, hipStream_t s)
{
    if constexpr (W >= kWideWidth) {
        const int nb = bwd_blocks(n_s);
        const int64_t per = ((n_s + 15) / 16 + nb - 1) / nb;
        constexpr size_t lds = WideLdsLp<IN, W, D>::BYTES;
        const hipError_t e = set_lds_lp(k_mlp_wide_bwd_lp<IN, W, D, P>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_mlp_wide_bwd_lp<IN, W, D, P>), dim3((uint32_t)nb), dim3(64 * kWideWavesLp), lds, s, w,
                           (const float2*)y, (const float4*)sc, (const float4*)dout, n_s, per, (float2*)dy, partial);
        return hipGetLastError();
    } else {
        const size_t lds = bwd_lds_lp<IN, W, D, P>();
        auto kern = k_mlp_bwd_lp<IN, W, D, P>;
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((uint32_t)bwd_blocks(n_s)), dim3(64 * kBwdWaves), lds, s, w, (const float2*)y,
                           (const float4*)dout, n_s, (float2*)dy, partial);
        return hipGetLastError();
    }
}

template <int IN, int W, int D, class P>
hipError_t fwd_lp_batch(const MlpWork* work, int n_blocks, const float* params, const float* y, float* sc, hipStream_t s)
{
    const size_t lds = fwd_lds_lp<IN, W, D, P>();
    hipError_t e = set_lds_lp(k_mlp_fwd_lp_batch<IN, W, D, P>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_mlp_fwd_lp_batch<IN, W, D, P>), dim3((uint32_t)n_blocks), dim3(256), lds, s, work, params,
                       (const float2*)y, (float4*)sc);
    return hipGetLastError();
}

template <int IN, int W, int D, class P>
hipError_t bwd_lp_batch(const MlpWork* work, int n_blocks, const float* params, const float* y, const float* dout,
                        const float* sc, float* dy, float* partial, int64_t slot_stride, hipStream_t s)
{
    if constexpr (W >= kWideWidth) {
        constexpr size_t lds = WideLdsLp<IN, W, D>::BYTES;
        const hipError_t e = set_lds_lp(k_mlp_wide_bwd_lp_batch<IN, W, D, P>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_mlp_wide_bwd_lp_batch<IN, W, D, P>), dim3((uint32_t)n_blocks), dim3(64 * kWideWavesLp), lds,
                           s, work, params, y, (const float4*)sc, (const float4*)dout, (float2*)dy, partial, slot_stride);
        return hipGetLastError();
    } else {
        const size_t lds = bwd_lds_lp<IN, W, D, P>();
        auto kern = k_mlp_bwd_lp_batch<IN, W, D, P>;
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((uint32_t)n_blocks), dim3(64 * kBwdWaves), lds, s, work, params,
                           (const float2*)y, (const float4*)dout, (float2*)dy, partial, slot_stride);
        return hipGetLastError();
    }
}

#define PRENOM_FOR_EACH_MLP_LP(X) \
    X(16, 32, 1) \
    X(16, 32, 2) \
    X(16, 64, 1) \
    X(16, 64, 2) \
    X(16, 128, 1) \
    X(16, 128, 2) \
    X(24, 32, 1) \
    X(24, 32, 2) \
    X(24, 64, 1) \
    X(24, 64, 2) \
    X(24, 128, 1) \
    X(24, 128, 2) \
    X(32, 32, 1) \
    X(32, 32, 2) \
    X(32, 64, 1) \
    X(32, 64, 2) \
    X(32, 128, 1) \
    X(32, 128, 2)

template <class P>
hipError_t fwd_dispatch(const MlpShape& m, const float* w, const float* y, int64_t n_s, float* sc, hipStream_t s)
{
#define X(I, Wd, Dp) \
    if (m.in_dim == I && m.width == Wd && m.hidden == Dp) return fwd_lp<I, Wd, Dp, P>(w, y, n_s, sc, s);
    PRENOM_FOR_EACH_MLP_LP(X)
#undef X
    return hipErrorInvalidValue;
}

template <class P>
hipError_t bwd_dispatch(const MlpShape& m, const float* w, const float* y, const float* dout, const float* sc,
                        int64_t n_s, float* dy, float* partial, hipStream_t s)
{
#define X(I, Wd, Dp)                                        \
    if (m.in_dim == I && m.width == Wd && m.hidden == Dp) \
        return bwd_lp<I, Wd, Dp, P>(w, y, dout, sc, n_s, dy, partial, s);
    PRENOM_FOR_EACH_MLP_LP(X)
#undef X
    return hipErrorInvalidValue;
}

template <class P>
hipError_t fwd_batch_dispatch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params, const float* y,
                              float* sc, hipStream_t s)
{
#define X(I, Wd, Dp)                                        \
    if (m.in_dim == I && m.width == Wd && m.hidden == Dp) \
        return fwd_lp_batch<I, Wd, Dp, P>(work, n_blocks, params, y, sc, s);
    PRENOM_FOR_EACH_MLP_LP(X)
#undef X
    return hipErrorInvalidValue;
}

template <class P>
hipError_t bwd_batch_dispatch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params,
                              const float* y, const float* dout, const float* sc, float* dy, float* partial,
                              int64_t slot_stride, hipStream_t s)
{
#define X(I, Wd, Dp)                                                                                     \
    if (m.in_dim == I && m.width == Wd && m.hidden == Dp)                                              \
        return bwd_lp_batch<I, Wd, Dp, P>(work, n_blocks, params, y, dout, sc, dy, partial, slot_stride, s);
    PRENOM_FOR_EACH_MLP_LP(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_mlp_fwd_lp(const MlpShape& m, const float* w, const float* y, int64_t n_s, float* sc, hipStream_t s)
{
    if (n_s == 0) return hipSuccess;
    if (m.dtype == PRENOM_BF16) return fwd_dispatch<Bf16Op>(m, w, y, n_s, sc, s);
    if (m.dtype == PRENOM_F16) return fwd_dispatch<F16Op>(m, w, y, n_s, sc, s);
    return hipErrorInvalidValue;
}

hipError_t launch_mlp_bwd_lp(const MlpShape& m, const float* w, const float* y, const float* dout, const float* sc,
                             int64_t n_s, float* dy, float* partial, hipStream_t s)
{
    if (n_s == 0) return hipSuccess;
    if (m.dtype == PRENOM_BF16) return bwd_dispatch<Bf16Op>(m, w, y, dout, sc, n_s, dy, partial, s);
    if (m.dtype == PRENOM_F16) return bwd_dispatch<F16Op>(m, w, y, dout, sc, n_s, dy, partial, s);
    return hipErrorInvalidValue;
}

hipError_t launch_mlp_fwd_lp_batch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params,
                                   const float* y, float* sc, hipStream_t s)
{
    if (n_blocks == 0) return hipSuccess;
    if (m.dtype == PRENOM_BF16) return fwd_batch_dispatch<Bf16Op>(m, work, n_blocks, params, y, sc, s);
    if (m.dtype == PRENOM_F16) return fwd_batch_dispatch<F16Op>(m, work, n_blocks, params, y, sc, s);
    return hipErrorInvalidValue;
}

hipError_t launch_mlp_bwd_lp_batch(const MlpShape& m, const MlpWork* work, int n_blocks, const float* params,
                                   const float* y, const float* dout, const float* sc, float* dy, float* partial,
                                   int64_t slot_stride, hipStream_t s)
{
    if (n_blocks == 0) return hipSuccess;
    if (m.dtype == PRENOM_BF16)
        return bwd_batch_dispatch<Bf16Op>(m, work, n_blocks, params, y, dout, sc, dy, partial, slot_stride, s);
    if (m.dtype == PRENOM_F16)
        return bwd_batch_dispatch<F16Op>(m, work, n_blocks, params, y, dout, sc, dy, partial, slot_stride, s);
    return hipErrorInvalidValue;
}

}  // namespace prenom
