// layer_kernels.hip -- MLP layers with both operands in MFMA fragment order,
// read from the L2 straight into registers: fp32 policies and critics, and
// bf16 ones on small batches.
//
// An fp32 value is carried as three bf16 planes, x = x0 + 2^-8 x1 + 2^-16 x2:
// x0 the value rounded to bf16, x1 the remainder (scaled) rounded, x2 the rest
// (8 + 8 + 8 significant bits).  With the scales every finite fp32 value,
// subnormal or not, is its planes' sum exactly; planes of the remainders as they
// are would leave bf16's range below 2^-110.  A product is eight plane products;
// the ninth, x2 w2, is below 2^-32 of it (2^-30 where one factor is subnormal).
// Products of equal scale 2^-8d have an accumulator of their own (d = 0 .. 3),
// joined at the end (join_sums), so that the leading ones are rounded once per
// 16 inputs and the others count fully.  Against float64, fp32 S15 at 64 to 8192
// envs: means 1.3e-7 to 1.8e-7 off by norm (fp32 MFMA kernels 5.0e-7 to 5.2e-7,
// six products without scales 2.1e-7 to 2.3e-7); outputs of a single product at
// most 2^-24 off (with six, 1e-7; 1e-4 and more for operands below 1e-36).
// Eight v_mfma_f32_32x32x16_bf16 take 256 cycles where the eight
// v_mfma_f32_32x32x2_f32 of the same 16 k take 512.  A sum that is not finite
// is formed again with fp32 products (fix_sums), so that infinities, NaNs and
// overflows come out as in fp32.
//
// Layout: activations and weights in 1 KB blocks, one per (tile of 32 envs or
// output features, 16 inputs, plane): lane l = 32 h + r holds inputs 16 s +
// 8 h .. +7 of row r, the operand of one MFMA as 16 consecutive bytes.  For
// one plane this is frag_index.
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "launch.h"
#include "sampling.h"

namespace im {

constexpr float BF16_MAX = 3.38953139e38f, FP32_MAX = 3.402823466e38f;

constexpr float PLANE = 0x1p-8f;     // scale of a plane against the one before

// The bf16 planes of N values, packed in pairs (the even one in the low half).
// Values that round to infinity take the truncated leading plane (their second
// plane then clamped to the type's largest value, the third holds what is left),
// infinities and NaNs are carried by it alone.
template <int P, int N>
__device__ __forceinline__ void split_planes(const float (&v)[N], uint32_t (&o)[P][N / 2])
{
#pragma unroll
    for (int i = 0; i < N / 2; ++i) o[0][i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    if constexpr (P == 3) {
        float mx = 0.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) mx = fmaxf(mx, fabsf(v[i]));
        const bool big = __any(!(mx <= BF16_MAX));
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            float hi[2] = {__uint_as_float(o[0][i] << 16), __uint_as_float(o[0][i] & 0xFFFF0000u)};
            float rest[2], mid[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) rest[q] = mid[q] = (v[2 * i + q] - hi[q]) * 256.0f;
            if (big) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float x = v[2 * i + q];
                    if (fabsf(x) > BF16_MAX) {
                        const bool fin = fabsf(x) <= FP32_MAX;
                        if (fin) hi[q] = __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
                        rest[q] = fin ? (x - hi[q]) * 256.0f : 0.0f;
                        mid[q] = fminf(fmaxf(rest[q], -BF16_MAX), BF16_MAX);
                    }
                }
                o[0][i] = (__float_as_uint(hi[0]) >> 16) | (__float_as_uint(hi[1]) & 0xFFFF0000u);
            }
            o[1][i] = pack_bf16x2(mid[0], mid[1]);
            o[2][i] = pack_bf16x2((rest[0] - __uint_as_float(o[1][i] << 16)) * 256.0f,
                                  (rest[1] - __uint_as_float(o[1][i] & 0xFFFF0000u)) * 256.0f);
        }
    }
}

// The fp32 value of three planes (exact).
__device__ __forceinline__ float join_planes(float x0, float x1, float x2)
{
    return fmaf(x2, PLANE * PLANE, fmaf(x1, PLANE, x0));
}

// Plane products by accumulator: NG accumulators, product (weight plane,
// input plane) into accumulator d, the sum of the two; in an order that
// returns to an accumulator as late as possible.
template <int P>
struct PlaneProducts;
template <>
struct PlaneProducts<1> {
    static constexpr int NG = 1, N = 1, W[1] = {0}, X[1] = {0};
};
template <>
struct PlaneProducts<3> {
    static constexpr int NG = 4, N = 8, W[8] = {2, 2, 1, 0, 1, 1, 0, 0}, X[8] = {1, 0, 0, 0, 2, 1, 1, 2};
};

// The sums of the accumulators of equal scale.
template <int NG>
__device__ __forceinline__ float join_sums(const float (&a)[NG])
{
    float s = a[NG - 1];
#pragma unroll
    for (int d = NG - 2; d >= 0; --d) s = fmaf(s, PLANE, a[d]);
    return s;
}

// Sums v (lane: env l & 31, register 4 grp + q: feature 8 grp + 4 (l >> 5) + q)
// of tile (mt, nt) over the 16-input steps k0 .. k1-1 that are not finite, again
// with fp32 products (v_mfma_f32_32x32x2_f32 on the planes' values), as one pass of
// the whole tile: a wave pays 0.3 us per 16 inputs however many of its sums are
// affected.  The others keep their value, so that a row does not depend on the
// rows beside it.  S15, 64 / 4096 envs, 23 / 67 us a call: 30 / 120 us with an
// infinity in one env's observation, 30 / 137 with one in every env's (each sum by
// one lane, term by term: 3.6 to 9 ms).
__device__ __forceinline__ void fix_sums(const LayerNet &a, int mt, int64_t nt, int k0, int k1, int lane,
                                         f32x16_t &v)
{
    bool bad = false;
#pragma unroll
    for (int q = 0; q < 16; ++q) bad = bad || !(fabsf(v[q]) <= FP32_MAX);
    if (!__any(bad)) return;
    struct Step {
        u32x4_t w[3], x[3];
    };
    auto load = [&](int s, Step &t) {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            t.w[p] = *((const u32x4_t *)(a.w + (((int64_t)mt * a.K16 + s) * 3 + p) * 512) + lane);
            t.x[p] = *((const u32x4_t *)(a.x + ((nt * a.K16 + s) * 3 + p) * 512) + lane);
        }
    };
    auto value = [](const u32x4_t (&t)[3], int i) {
        float f[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) f[p] = __uint_as_float(i & 1 ? t[p][i >> 1] & 0xFFFF0000u : t[p][i >> 1] << 16);
        return join_planes(f[0], f[1], f[2]);
    };
    f32x16_t c;
#pragma unroll
    for (int q = 0; q < 16; ++q) c[q] = 0.0f;
    Step cur, nxt;
    load(k0, nxt);      // (k0 < k1: the sums of no inputs are zero)
#pragma unroll 1
    for (int s = k0; s < k1; ++s) {
        cur = nxt;
        load(s + 1 < k1 ? s + 1 : s, nxt);
#pragma unroll
        for (int i = 0; i < 8; ++i)     // inputs 16 s + i of the lower half wave, 16 s + 8 + i of the upper
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(value(cur.w, i), value(cur.x, i), c, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = fabsf(v[q]) <= FP32_MAX ? v[q] : c[q];
}

// The observation [D][ld] (env fastest) into operand blocks, a wavefront per
// (tile of 32 envs, 16 inputs): inputs past D are zero, envs past N repeat the
// last.  Once per call: the first layer's blocks, each converting its envs
// anew with 4-byte loads, took 37 us for 4096 envs of 226 inputs in fp32,
// against 5.4 us here and 21.6 us for the layer.
template <int P>
__global__ __launch_bounds__(256) void stage_planes_kernel(const float *__restrict__ obs, int64_t ld, int D,
                                                           int64_t N, int K16, uint16_t *__restrict__ x)
{
    const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t nt = b / K16;
    const int s = (int)(b % K16);
    if (nt * 32 >= N) return;
    const int64_t n = nt * 32 + (lane & 31), e = n < N ? n : N - 1;
    const int k0 = 16 * s + 8 * (lane >> 5);
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int k = k0 + q;
        const float t = obs[(int64_t)(k < D ? k : D - 1) * ld + e];
        v[q] = k < D ? t : 0.0f;
    }
    uint32_t o[P][4];
    split_planes<P, 8>(v, o);
#pragma unroll
    for (int p = 0; p < P; ++p)
        *((u32x4_t *)(x + (b * P + p) * 512) + lane) = u32x4_t{o[p][0], o[p][1], o[p][2], o[p][3]};
}

// fp32 weights [M][16 K16] (row-major, M a multiple of 32) into operand blocks,
// a wavefront per (tile of 32 rows, 16 inputs).  Once per network.
__global__ __launch_bounds__(256) void pack_planes_kernel(const float *__restrict__ src, int M, int K16,
                                                          uint16_t *__restrict__ w)
{
    const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= (int64_t)(M / 32) * K16) return;
    const int lane = threadIdx.x & 63;
    const float *q = src + ((b / K16) * 32 + (lane & 31)) * 16 * K16 + 16 * (b % K16) + 8 * (lane >> 5);
    float v[8];
    uint32_t o[3][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = q[i];
    split_planes<3, 8>(v, o);
#pragma unroll
    for (int p = 0; p < 3; ++p)
        *((u32x4_t *)(w + (b * 3 + p) * 512) + lane) = u32x4_t{o[p][0], o[p][1], o[p][2], o[p][3]};
}

// acc += W[32][k] X[32][k]^T of weight tile mt and env tile nt over the 16-input
// steps k0 .. k1-1.  U steps of operands are loaded at a time, two such sets in
// turn, so that one is in flight while the other is multiplied (steps past the
// end of a set load the last one again).
template <int P, int U>
__device__ __forceinline__ void layer_mma(const LayerNet &a, int mt, int64_t nt, int k0, int k1,
                                          int lane, f32x16_t (&acc)[PlaneProducts<P>::NG])
{
    using Prod = PlaneProducts<P>;
    struct Set {
        u32x4_t w[U][P], x[U][P];
    };
    auto load = [&](int k, Set &t) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = k + u < k1 ? k + u : k1 - 1;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                t.w[u][p] = *((const u32x4_t *)(a.w + (((int64_t)mt * a.K16 + s) * P + p) * 512) + lane);
                t.x[u][p] = *((const u32x4_t *)(a.x + ((nt * a.K16 + s) * P + p) * 512) + lane);
            }
        }
    };
    auto mma = [&](int k, const Set &t) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k + u >= k1) break;
#pragma unroll
            for (int c = 0; c < Prod::N; ++c) {
                f32x16_t &t16 = acc[Prod::W[c] + Prod::X[c]];
                t16 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8_t, t.w[u][Prod::W[c]]),
                    __builtin_bit_cast(bf16x8_t, t.x[u][Prod::X[c]]), t16, 0, 0, 0);
            }
        }
    };
    // (scheduling barriers keep the loads ahead of the products)
    if (k0 >= k1) return;
    Set ta, tb;
    load(k0, ta);
    for (int k = k0; k < k1; k += 2 * U) {
        if (k + U < k1) load(k + U, tb);
        __builtin_amdgcn_sched_barrier(0);
        mma(k, ta);
        if (k + 2 * U < k1) load(k + 2 * U, ta);
        __builtin_amdgcn_sched_barrier(0);
        mma(k + U, tb);
    }
}

// The fp32 sums of a tile over the steps k0 .. k1-1.
template <int U>
__device__ __forceinline__ f32x16_t plane_sums(const LayerNet &a, int mt, int64_t nt, int k0, int k1, int lane)
{
    f32x16_t acc[4], v;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[d][q] = 0.0f;
    layer_mma<3, U>(a, mt, nt, k0, k1, lane, acc);
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = join_sums<4>({acc[0][q], acc[1][q], acc[2][q], acc[3][q]});
    fix_sums(a, mt, nt, k0, k1, lane, v);
    return v;
}

// The sums v of tile (mt, nt) (layout: fix_sums), bias added, to the layer's
// output: ReLU, planes.
template <int P>
__device__ __forceinline__ void finish_tile(const LayerNet &a, int mt, int64_t nt, int lane, float (&v)[16])
{
    if constexpr (P == 3)
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = fmaxf(v[q], 0.0f);
    uint32_t o[P][8];
    split_planes<P, 16>(v, o);
    if constexpr (P == 1)
#pragma unroll
        for (int q = 0; q < 8; ++q) o[0][q] = relu_bf16x2(o[0][q]);
    // the half waves trade groups: lanes of half 0 keep features 0-7 and
    // 16-23 of the tile, half 1 features 8-15 and 24-31, each 16 bytes of
    // its lane in the blocks of the tile's two 16-feature steps
#pragma unroll
    for (int pl = 0; pl < P; ++pl) {
        uint16_t *y = a.y + ((nt * (a.M / 16) + 2 * mt) * P + pl) * 512 + 8 * lane;
        const auto a0 = __builtin_amdgcn_permlane32_swap(o[pl][0], o[pl][2], false, false);
        const auto a1 = __builtin_amdgcn_permlane32_swap(o[pl][1], o[pl][3], false, false);
        const auto b0 = __builtin_amdgcn_permlane32_swap(o[pl][4], o[pl][6], false, false);
        const auto b1 = __builtin_amdgcn_permlane32_swap(o[pl][5], o[pl][7], false, false);
        *(u32x4_t *)y = u32x4_t{a0[0], a1[0], a0[1], a1[1]};
        *(u32x4_t *)(y + P * 512) = u32x4_t{b0[0], b1[0], b0[1], b1[1]};
    }
}

// Hidden layer, y = ReLU(W x + b), fp32, on few envs: a block is one tile of 32
// features x 32 envs, its 8 waves split the inputs; no operand is staged, the
// partial tiles meet in LDS and the first wave adds them in wave order.
template <int U>
__global__ __launch_bounds__(512, 1) void layer_small_kernel(LayerPair p)
{
    constexpr int WK = 8;
    __shared__ f32x4_t red[WK][4][64];
    int id = xcd_order(blockIdx.x, gridDim.x);
    const bool second = id >= p.blocks0;
    if (second) id -= p.blocks0;
    const LayerNet a = second ? p.a[1] : p.a[0];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mt = id % (a.M / 32);
    const int64_t nt = id / (a.M / 32);
    float4 bias[4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
        bias[grp] = *(const float4 *)(a.bias + 32 * mt + 8 * grp + 4 * (lane >> 5));
    const f32x16_t part = plane_sums<U>(a, mt, nt, wave * a.K16 / WK, (wave + 1) * a.K16 / WK, lane);
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
        red[wave][grp][lane] = f32x4_t{part[4 * grp], part[4 * grp + 1], part[4 * grp + 2], part[4 * grp + 3]};
    __syncthreads();
    if (wave > 0) return;
    float v[16];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
        f32x4_t s = red[0][grp][lane];
#pragma unroll
        for (int k = 1; k < WK; ++k) s += red[k][grp][lane];
        v[4 * grp] = s[0] + bias[grp].x;
        v[4 * grp + 1] = s[1] + bias[grp].y;
        v[4 * grp + 2] = s[2] + bias[grp].z;
        v[4 * grp + 3] = s[3] + bias[grp].w;
    }
    finish_tile<3>(a, mt, nt, lane, v);
}

// The same in bf16, a wave (and block) per tile: the sums start at the bias and
// take the inputs in order, as in the one-launch kernel, whose bits these are;
// a row's result does not depend on the batch it comes in.  16 steps of operands
// (32 KB) in flight at a time, two such sets.
__global__ __launch_bounds__(64, 1) void layer_small_bf16_kernel(LayerPair p)
{
    int id = xcd_order(blockIdx.x, gridDim.x);
    const bool second = id >= p.blocks0;
    if (second) id -= p.blocks0;
    const LayerNet a = second ? p.a[1] : p.a[0];
    const int lane = threadIdx.x;
    const int mt = id % (a.M / 32);
    const int64_t nt = id / (a.M / 32);
    f32x16_t acc[1];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
        const float4 b = *(const float4 *)(a.bias + 32 * mt + 8 * grp + 4 * (lane >> 5));
        acc[0][4 * grp] = b.x;
        acc[0][4 * grp + 1] = b.y;
        acc[0][4 * grp + 2] = b.z;
        acc[0][4 * grp + 3] = b.w;
    }
    layer_mma<1, 16>(a, mt, nt, 0, a.K16, lane, acc);
    float v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = acc[0][q];
    finish_tile<1>(a, mt, nt, lane, v);
}

// Order of a phase of the next kernel: its NM products with its NR fragment
// reads spread over the first two thirds of them and its NW other accesses
// (MASK: LDS writes or global loads) over the last half.  A wave issues in
// order, and with one wave per SIMD a run of reads would keep the matrix core
// idle for as long as the LDS takes to accept them.
template <int MASK, int NM, int NR, int NW, int K = 0>
__device__ __forceinline__ void phase_order()
{
    if constexpr (K < NM) {
        constexpr auto least = [](int a, int b) { return a < b ? a : b; };
        constexpr auto most = [](int a, int b) { return a > b ? a : b; };
        constexpr int r0 = least(NR, K * NR * 3 / (2 * NM));
        constexpr int r1 = K + 1 == NM ? NR : least(NR, (K + 1) * NR * 3 / (2 * NM));
        constexpr int w0 = most(0, (2 * K - NM) * NW / NM), w1 = most(0, (2 * (K + 1) - NM) * NW / NM);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (r1 > r0) __builtin_amdgcn_sched_group_barrier(0x100, r1 - r0, 0);
        if constexpr (w1 > w0) __builtin_amdgcn_sched_group_barrier(MASK, w1 - w0, 0);
        phase_order<MASK, NM, NR, NW, K + 1>();
    } else {
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The same on many envs, fp32: tiles of 32 BT features x 32 BT envs, 2 BT waves
// of BT/2 x 1 MFMA tiles, each of which brings in one of the 2 BT operand tiles.
// Two 16-input steps of operand blocks (a block is 1 KB of consecutive bytes, in
// memory as in LDS, and a fragment read its 16 bytes per lane: no bank
// conflicts) are staged at a time, two LDS buffers, the loads NS stages ahead in
// as many sets of registers.
// S15, 4096 envs, layers 226-1024 and 1024-512: 20.3 and 34.3 us (fp32 MFMA
// kernels on 64 x 64 tiles 29.5 and 45.7; six plane products, one accumulator
// for the smaller ones, 19.8 and 31.7); at 16384 envs 83 and 126 us, the matrix
// cores busy for 41 and 82 of them.  With four waves on the 128 x 128 tile the
// accumulators leave no registers for the operands (700 bytes of spills).  With
// six products, the reads ahead of the products instead of between them took 10%
// longer; operands straight from the L2 on 64 x 128 tiles, the waves splitting the
// inputs, were no faster at 16384 envs.
template <int BT>
__global__ __launch_bounds__(128 * BT, (BT == 2 ? 2 : 1)) void layer_kernel(LayerPair p)
{
    using Prod = PlaneProducts<3>;
    constexpr int P = 3, TM = BT / 2, TN = 1, BL = 2 * BT * 2 * P;  // blocks per stage
    constexpr int PW = 2 * P;                 // by wave: those of one of the 2 BT tiles
    constexpr int NS = BT == 4 ? 2 : 4;       // register sets: stages in flight
    __shared__ __attribute__((aligned(16))) uint16_t lds[2][BL * 512];
    int id = xcd_order(blockIdx.x, gridDim.x);
    const bool second = id >= p.blocks0;
    if (second) id -= p.blocks0;
    const LayerNet a = second ? p.a[1] : p.a[0];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mblocks = a.M / (32 * BT);
    const int mt0 = (id % mblocks) * BT;
    const int64_t nt0 = (int64_t)(id / mblocks) * BT;
    const int wm = wave & 1, wn = wave >> 1;
    const int nk = a.K16 / 2;       // stages
    // this wave's blocks of a stage: the consecutive ones of one tile
    const uint16_t *src = (wave < BT ? a.w + (int64_t)(mt0 + wave) * a.K16 * P * 512
                                     : a.x + (nt0 + wave - BT) * a.K16 * P * 512) + 8 * lane;
    u32x4_t rs[NS][PW];
    auto load = [&](int kt, u32x4_t (&r)[PW]) {
        const int k = kt < nk ? kt : nk - 1;
#pragma unroll
        for (int c = 0; c < PW; ++c) r[c] = *(const u32x4_t *)(src + ((int64_t)k * PW + c) * 512);
    };
    auto store = [&](int buf, const u32x4_t (&r)[PW]) {
#pragma unroll
        for (int c = 0; c < PW; ++c) *((u32x4_t *)(lds[buf] + (wave * PW + c) * 512) + lane) = r[c];
    };
    f32x16_t acc[Prod::NG][TM][TN];
#pragma unroll
    for (int l = 0; l < Prod::NG; ++l)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[l][i][j][q] = 0.0f;
    struct Frags {
        bf16x8_t w[TM][P], x[TN][P];
    };
    auto read = [&](int buf, int u, Frags &f) {
#pragma unroll
        for (int pl = P - 1; pl >= 0; --pl) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                f.w[i][pl] = *((const bf16x8_t *)(lds[buf] + (((wm * TM + i) * 2 + u) * P + pl) * 512) + lane);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                f.x[j][pl] = *((const bf16x8_t *)(lds[buf] + (((BT + wn * TN + j) * 2 + u) * P + pl) * 512) + lane);
        }
    };
    auto mma = [&](const Frags &f) {
#pragma unroll
        for (int c = 0; c < Prod::N; ++c)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    f32x16_t &t = acc[Prod::W[c] + Prod::X[c]][i][j];
                    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[i][Prod::W[c]], f.x[j][Prod::X[c]], t, 0, 0, 0);
                }
    };
    constexpr int NM = TM * TN * Prod::N, NR = (TM + TN) * P;
    // stage kt in buffer kt & 1, the next one on its way in r: its second step
    // is read before the products of the first; the next stage is written
    // (its buffer was last read before the previous barrier), and its first
    // step read before the products of the second
    Frags f0, f1;
    auto stage = [&](int kt, int buf, u32x4_t (&r)[PW]) {
        read(buf, 1, f1);
        mma(f0);
        store(buf ^ 1, r);
        phase_order<0x200, NM, NR, PW>();
        __syncthreads();
        read(buf ^ 1, 0, f0);
        mma(f1);
        load(kt + 1 + NS, r);
        phase_order<0x020, NM, NR, PW>();
    };
#pragma unroll
    for (int i = 0; i < NS; ++i) load(i, rs[i]);
    store(0, rs[0]);
    load(NS, rs[0]);
    __syncthreads();
    read(0, 0, f0);
    for (int kt = 0;;) {        // nk is even
        stage(kt, 0, rs[1]);
        stage(kt + 1, 1, rs[2 % NS]);
        if ((kt += 2) >= nk) break;
        if constexpr (NS == 4) {
            stage(kt, 0, rs[3]);
            stage(kt + 1, 1, rs[0]);
            if ((kt += 2) >= nk) break;
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int mt = mt0 + wm * TM + i;
        float4 bias[4];
#pragma unroll
        for (int grp = 0; grp < 4; ++grp)
            bias[grp] = *(const float4 *)(a.bias + 32 * mt + 8 * grp + 4 * (lane >> 5));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t nt = nt0 + wn * TN + j;
            if (nt * 32 >= a.N) continue;
            f32x16_t sum;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                float t[Prod::NG];
#pragma unroll
                for (int d = 0; d < Prod::NG; ++d) t[d] = acc[d][i][j][q];
                sum[q] = join_sums<Prod::NG>(t);
            }
            fix_sums(a, mt, nt, 0, a.K16, lane, sum);
            float v[16];
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                v[4 * grp] = sum[4 * grp] + bias[grp].x;
                v[4 * grp + 1] = sum[4 * grp + 1] + bias[grp].y;
                v[4 * grp + 2] = sum[4 * grp + 2] + bias[grp].z;
                v[4 * grp + 3] = sum[4 * grp + 3] + bias[grp].w;
            }
            finish_tile<P>(a, mt, nt, lane, v);
        }
    }
}

// Last layers: blocks below nb_policy sample the actions of 32 envs each (the
// layer's 32 MT padded actions, the waves splitting the inputs), the rest form
// the values of 32 envs each (the fp32 head on the planes' values, 8 waves
// splitting the inputs, partials added in wave order).  bf16: the slices and the
// order of the sums are those of the one-launch kernel, bit for bit.
template <int P, int MT>
__global__ __launch_bounds__(512, P == 3 && MT == 1 ? 4 : 1) void layer_out_kernel(LayerNet a, GemmArgs g, LayerHead v, int nb_policy)
{
    // KS slices of the inputs by MT action tiles.  fp32: 8 waves, a wave takes
    // TM tiles, one after the other (the accumulators of several at once would
    // not fit beside the operands in flight; four tiles by eight slices would not
    // fit in LDS).  bf16: one tile a wave, 6 or 4 waves at three and four tiles.
    // One action tile in fp32 loads a step at a time, which leaves room for two
    // blocks a CU (128 registers): 65536 envs of 256 inputs 40 -> 29 us.
    constexpr int MP = 32 * MT, WK = 8, KS = P == 3 ? (MT == 4 ? 4 : 8) : (MT == 4 ? 1 : (MT == 3 ? 2 : 8 / MT));
    constexpr int TM = P == 3 ? MT * KS / 8 : 1;
    __shared__ __attribute__((aligned(16))) float lds[(KS + 2) * 32 * MP + 32 * 33];
    __shared__ float sig[128], sbias[128], slp0;
    __shared__ uint32_t senv[32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, r = lane & 31;
    if ((int)blockIdx.x >= nb_policy) {
        const int64_t nt = (int)blockIdx.x - nb_policy, n = nt * 32 + r;
        if constexpr (P == 1) {
            // a wave's inputs in order, chunks of 8 (both half waves alike)
            const int per = v.K16 / 4;
            float acc = 0.0f;
#pragma unroll 4
            for (int c = wave * per; c < (wave + 1) * per; ++c) {
                const u32x4_t x = *((const u32x4_t *)(v.x + (nt * v.K16 + (c >> 1)) * 512) + 32 * (c & 1) + r);
                const float *w = v.head + 8 * c;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc += w[2 * i] * __uint_as_float(x[i] << 16);
                    acc += w[2 * i + 1] * __uint_as_float(x[i] & 0xFFFF0000u);
                }
            }
            if (h == 0) lds[wave * 32 + r] = acc;
            __syncthreads();
            if (tid < 32 && n < v.N) {
                float s = v.head[16 * v.K16];
#pragma unroll
                for (int k = 0; k < WK; ++k) s += lds[k * 32 + tid];
                v.value[n] = s;
            }
            return;
        }
        float acc = 0.0f;
#pragma unroll 2
        for (int s = wave * v.K16 / WK; s < (wave + 1) * v.K16 / WK; ++s) {
            const u32x4_t *x = (const u32x4_t *)(v.x + ((nt * v.K16 + s) * 3) * 512) + lane;
            const float *w = v.head + 16 * s + 8 * h;
            u32x4_t q[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) q[p] = x[64 * p];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc += w[2 * i] * join_planes(__uint_as_float(q[0][i] << 16), __uint_as_float(q[1][i] << 16),
                                              __uint_as_float(q[2][i] << 16));
                acc += w[2 * i + 1] * join_planes(__uint_as_float(q[0][i] & 0xFFFF0000u),
                                                  __uint_as_float(q[1][i] & 0xFFFF0000u),
                                                  __uint_as_float(q[2][i] & 0xFFFF0000u));
            }
        }
        lds[(2 * wave + h) * 32 + r] = acc;
        __syncthreads();
        if (tid < 32 && n < v.N) {
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k < 2 * WK; ++k) s += lds[k * 32 + tid];
            v.value[n] = s + v.head[16 * v.K16];
        }
        return;
    }
    const int A = g.A;
    const int64_t n0 = g.env0 + (int64_t)blockIdx.x * 32;
    const int64_t nv = g.N - n0 < 32 ? g.N - n0 : 32;
    float ls = 0.0f, bv = 0.0f;
    if (tid < A) {
        ls = g.log_std[tid];
        bv = g.bias[tid];
    }
    if (tid >= 256 && tid < 256 + nv) senv[tid - 256] = g.env_n[n0 + tid - 256];
    const int ksl = P == 3 ? wave % KS : wave / MT, mt0 = P == 3 ? wave / KS * TM : wave % MT;
    if (P == 3 || wave < MT * KS) {
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            f32x16_t v16;
            if constexpr (P == 3) {
                v16 = plane_sums<MT == 1 ? 1 : 2>(a, mt0 + t, blockIdx.x, ksl * a.K16 / KS, (ksl + 1) * a.K16 / KS, lane);
            } else {
                f32x16_t acc[1];
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[0][q] = 0.0f;
                const int nks = a.K16 / 4;      // slices of whole K steps of 64
                layer_mma<1, 8>(a, mt0, blockIdx.x, 4 * (ksl * nks / KS), 4 * ((ksl + 1) * nks / KS), lane, acc);
                v16 = acc[0];
            }
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const int unit = (8 * (mt0 + t) + 2 * grp + h) ^ (r & 7);
                *(f32x4_t *)(lds + (ksl * 32 + r) * MP + 4 * unit) =
                    f32x4_t{v16[4 * grp], v16[4 * grp + 1], v16[4 * grp + 2], v16[4 * grp + 3]};
            }
        }
    }
    if (tid < 128) {
        sig[tid] = expf(ls);
        sbias[tid] = bv;
        if (tid >= 64) lds[KS * 32 * MP + tid - 64] = tid < A ? ls + HALF_LOG_2PI : 0.0f;
    }
    __syncthreads();
    if (tid < 64) {
        float c = (tid < A ? ls + HALF_LOG_2PI : 0.0f) + lds[KS * 32 * MP + tid];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
        if (tid == 0) slp0 = c;
    }
    __syncthreads();
    sample_rows<512, 32, MP, KS>(g, lds, sig, sbias, slp0, senv, n0, nv, tid);
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
// Tile of a hidden layer of M features and 16 K16 inputs on N envs (fp32; a
// bf16 network comes here with few envs only).  128 x 128 where that gives
// every CU a block; else layer_small_kernel while 2.3 us and its rounds of
// blocks, 2 + 0.08 K16 us each, cost less than the 5.2 + 0.18 K16 us of one block
// of 64 x 64; else 64 x 64.  Measured (us; small / 64 x 64 / 128 x 128), 1024
// features of 256 inputs: 256 envs 5.9 / 8.1 / 14.3, 512 envs 8.9 / 8.5 / 15.1,
// 1000 envs 15.6 / 10.3 / 15.1, 3000 envs 40 / 19.0 / 18.8, 4096 envs 52 / 23.7 /
// 20.3; 512 features of 1024 inputs: 512 envs 9.3 / 17.4 / 38, 1000 envs 16.4 /
// 18.4 / 39, 2048 envs 30 / 20.5 / 41, 4096 envs 57 / 34.3 / 45, 8192 envs 111 /
// 64.6 / 54.6.
enum { LAYER_SMALL = 0, LAYER_64, LAYER_128 };
static int layer_tile(const LayerNet &a, int planes, int n_cu)
{
    if (planes == 1) return LAYER_SMALL;
    const int64_t cu = n_cu > 0 ? n_cu : 1;
    if (a.M % 128 == 0 && (a.M / 128) * ((a.N + 127) / 128) >= cu) return LAYER_128;
    const int64_t rounds = ((int64_t)(a.M / 32) * ((a.N + 31) / 32) + cu - 1) / cu;
    return 230 + rounds * (200 + 8 * a.K16) <= 520 + 18 * a.K16 ? LAYER_SMALL : LAYER_64;
}

static hipError_t launch_layer_t(int planes, LayerPair p, int tile, hipStream_t s)
{
    const int t32 = tile == LAYER_128 ? 4 : (tile == LAYER_64 ? 2 : 1);      // 32-row tiles a side
    int64_t blocks[2] = {0, 0};
    for (int k = 0; k < p.n; ++k)
        blocks[k] = (int64_t)(p.a[k].M / (32 * t32)) * ((p.a[k].N + 32 * t32 - 1) / (32 * t32));
    if (blocks[0] + blocks[1] > 0x7FFFFFFF) return hipErrorInvalidValue;
    p.blocks0 = (int)blocks[0];
    const dim3 grid((unsigned)(blocks[0] + blocks[1]));
    if (planes == 1) hipLaunchKernelGGL(layer_small_bf16_kernel, grid, dim3(64), 0, s, p);
    else if (tile == LAYER_128) hipLaunchKernelGGL(layer_kernel<4>, grid, dim3(512), 0, s, p);
    else if (tile == LAYER_64) hipLaunchKernelGGL(layer_kernel<2>, grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL(layer_small_kernel<2>, grid, dim3(512), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_layers(int planes, const LayerNet *a, int n, int n_cu, hipStream_t s)
{
    for (int k = 0; k < n; ++k)
        if (a[k].N <= 0 || a[k].M <= 0 || a[k].M % 64 || a[k].K16 <= 0 || a[k].K16 % 4) return hipErrorInvalidValue;
    // one launch where both networks take the same tile (which a network's
    // results must not depend on: each is chosen for the network alone)
    const bool both = n == 2 && layer_tile(a[0], planes, n_cu) == layer_tile(a[1], planes, n_cu);
    for (int k = 0; k < n; k += both ? 2 : 1) {
        LayerPair p{};
        p.n = both ? 2 : 1;
        for (int q = 0; q < p.n; ++q) p.a[q] = a[k + q];
        const hipError_t e = launch_layer_t(planes, p, layer_tile(a[k], planes, n_cu), s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pack_planes(const float *src, int M, int K16, uint16_t *w, hipStream_t s)
{
    if (M <= 0 || M % 32 || K16 <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(pack_planes_kernel, dim3((unsigned)(((int64_t)(M / 32) * K16 + 3) / 4)), dim3(256), 0, s,
                       src, M, K16, w);
    return hipGetLastError();
}

hipError_t launch_stage_planes(int planes, const float *obs, int64_t ld, int D, int64_t N, int K16, uint16_t *x,
                               hipStream_t s)
{
    const int64_t blocks = ((N + 31) / 32 * K16 + 3) / 4;
    if (N <= 0 || K16 <= 0 || D <= 0 || blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    if (planes == 3) hipLaunchKernelGGL(stage_planes_kernel<3>, grid, dim3(256), 0, s, obs, ld, D, N, K16, x);
    else hipLaunchKernelGGL(stage_planes_kernel<1>, grid, dim3(256), 0, s, obs, ld, D, N, K16, x);
    return hipGetLastError();
}

hipError_t launch_layer_out(int planes, const LayerNet *a, const GemmArgs *g, const LayerHead *v, hipStream_t s)
{
    const int64_t np = a ? (g->N - g->env0 + 31) / 32 : 0, nv = v ? (v->N + 31) / 32 : 0;
    if (np + nv == 0) return hipSuccess;
    const int mt = a ? a->M / 32 : 1;
    if (a && (a->M % 32 || mt < 1 || mt > 4 || g->A > a->M || a->K16 <= 0)) return hipErrorInvalidValue;
    const LayerNet an = a ? *a : LayerNet{};
    const GemmArgs gn = a ? *g : GemmArgs{};
    const LayerHead vn = v ? *v : LayerHead{};
    const dim3 grid((unsigned)(np + nv));
#define IM_LO(P)                                                                                       \
    switch (mt) {                                                                                      \
        case 1: hipLaunchKernelGGL((layer_out_kernel<P, 1>), grid, dim3(512), 0, s, an, gn, vn, (int)np); break; \
        case 2: hipLaunchKernelGGL((layer_out_kernel<P, 2>), grid, dim3(512), 0, s, an, gn, vn, (int)np); break; \
        case 3: hipLaunchKernelGGL((layer_out_kernel<P, 3>), grid, dim3(512), 0, s, an, gn, vn, (int)np); break; \
        default: hipLaunchKernelGGL((layer_out_kernel<P, 4>), grid, dim3(512), 0, s, an, gn, vn, (int)np); break; \
    }
    if (planes == 3) {
        IM_LO(3)
    } else {
        IM_LO(1)
    }
#undef IM_LO
    return hipGetLastError();
}

}  // namespace im
