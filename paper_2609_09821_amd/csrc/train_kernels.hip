// train_kernels.hip -- the PPO update (the training loop's update_policy of
// Fig. 3) for bf16 actor-critic MLPs: minibatch gather from the rollout
// storage, forward and backward GEMMs on MFMA, the clipped-surrogate loss,
// deterministic gradient reductions, global-norm clip, KL-adaptive learning
// rate and Adam, all on the device with no host round trip.
//
// Layout: every activation and gradient is feature-major, [features][Mb]
// with the minibatch's samples contiguous (bf16), so the MFMA accumulator
// (one sample per lane, four consecutive features per register group) is
// stored without a transpose, and all three products of a layer
//   forward  Y^T  = W   X^T          (out x Mb)
//   backward dX^T = W^T dZ^T         (in x Mb, masked by the ReLU)
//   weights  dW   = dZ^T X           (out x in, reduced over the minibatch)
// are C[m][n] = sum_k A[m][k] B(k, n): A always has k contiguous (weights,
// transposed weights, dZ^T), B either k-major [k][n] (activations, gradients) or
// n-major [n][k] (X^T for the weight gradient).  The first two run on
// fgemm_kernel where the output width is a multiple of its 256 rows, the rest on
// tgemm_kernel.
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "launch.h"

namespace im {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4_v __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_v __attribute__((ext_vector_type(2)));
typedef short v4s_t __attribute__((ext_vector_type(4)));
#define IM_LDS3 __attribute__((address_space(3)))

// x plus the value DPP control CTRL brings in (0 where it brings none: lanes
// outside ROW_MASK, or shifted in from outside the row).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float x)
{
    const int t = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROW_MASK, 0xF, true);
    return x + __builtin_bit_cast(float, t);
}

// Sum of x over each group of W (16 or 32) consecutive lanes, aligned to W,
// returned in the group's last lane: an inclusive scan within each 16-lane
// row (DPP row shifts by 1, 2, 4, 8; lanes shifted in from outside the row
// read zero), then for W = 32 the total of the even row added into the odd
// row (row broadcast of lane 15).  The order of the additions is fixed.
template <int W>
__device__ __forceinline__ float lane_group_sum(float x)
{
    static_assert(W == 16 || W == 32, "lane group");
    x = dpp_add<0x111, 0xF>(x);     // row_shr:1
    x = dpp_add<0x112, 0xF>(x);     // row_shr:2
    x = dpp_add<0x114, 0xF>(x);     // row_shr:4
    x = dpp_add<0x118, 0xF>(x);     // row_shr:8
    if constexpr (W == 32)
        x = dpp_add<0x142, 0xA>(x); // row_bcast:15 into rows 1 and 3 (row mask 0b1010)
    return x;
}

// ---------------------------------------------------------------------------
// GEMM: tiles of BM = 64 WM rows by 256 columns (WM x 2 waves, each wave
// 64 x 128 = 2 x 4 MFMA 32x32x16 tiles).  WM = 4 (256 rows, 8 waves, 512
// threads) for weight gradients whose M is a multiple of 256, else WM = 2 (128
// rows, 4 waves): the other weight gradients, the actor's output layer, and the
// hidden layers that fgemm_kernel does not take.  K step 64, two LDS stages;
// loads of stage k+2 are in flight while stage k runs.  k-contiguous operands
// sit in LDS rows of 72 bf16 (144 bytes: fragment reads free of bank
// conflicts).  A k-major B tile is stored as it lies in memory, [64 k][256 n]
// in rows of 272 bf16, and its MFMA fragments are read with the LDS transpose
// read: in every 16-lane group, lane 4j+q addresses row k0+j, columns n0+4q..
// n0+4q+3, and lane l receives rows k0..k0+3 of column n0+l (two reads give the
// 8 consecutive k of a bf16 fragment; the 32-byte row shift of the padding keeps
// a group's four rows on distinct banks).  A split K (weight gradients: K = the
// minibatch) takes one block per tile and split.  All operands are zero-padded
// to whole tiles.
// ---------------------------------------------------------------------------
template <bool BT, int EPI, int WM>
__global__ __launch_bounds__(128 * WM) void tgemm_kernel(TGemmPair p)
{
    // this block's product, tile and K split: blocks of one XCD (dispatched
    // round robin over the 8) take consecutive (split, tile) numbers, so that
    // the tiles that share a B panel (or, split, a K range) share an L2
    int id = xcd_order(blockIdx.x, gridDim.x);
    const bool second = id >= p.blocks0;
    if (second) id -= p.blocks0;
    const TGemm g = second ? p.g[1] : p.g[0];
    // WM x 2 waves, each 64 x BN/2 (TN = BN/64 MFMA tiles across); tile BM x BN
    constexpr int NT = 128 * WM, BN = 256;
    constexpr int TN = BN / 64;
    constexpr int BM = 64 * WM, BK = 64, LDK = BK + 8;
    constexpr int LDN = BN + 16;                // k-major B rows (bf16)
    static_assert(BK * LDN <= BN * LDK + BK * 16, "stage size");
    constexpr int STAGE = BM * LDK + (BT ? BK * LDN : BN * LDK);
    __shared__ __attribute__((aligned(16))) uint16_t lds[2 * STAGE];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;   // wave: 64 x 64 of the tile
    const int mblocks = g.M / BM;
    const int tiles = mblocks * (g.N / BN);
    const int tile = id % tiles, split = id / tiles;
    const int64_t m0 = (int64_t)(tile % mblocks) * BM;
    const int64_t n0 = (int64_t)(tile / mblocks) * BN;
    const int kb = split * g.k_split;
    const int ke = kb + g.k_split < g.K ? kb + g.k_split : g.K;
    const int nk = (ke - kb) / BK;
    const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(
        (void *)g.A, (short)0, (int)g.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
        (void *)g.B, (short)0, (int)g.b_bytes, 0x00020000);

    // A: BM rows x 8 chunks of 16 bytes; B: BN rows x 8 chunks (n-major) or
    // 64 rows x BN/8 chunks of 8 samples (k-major)
    constexpr int AC = BM * 8 / NT, BC = BN * 8 / NT;
    constexpr int BQ = BN / 8;                  // k-major chunks per row
    uint32_t a_off[AC], b_off[BC];
#pragma unroll
    for (int c = 0; c < AC; ++c) {
        const int v = tid + c * NT;
        a_off[c] = (uint32_t)(((m0 + (v >> 3)) * g.lda + kb + (v & 7) * 8) * 2);
    }
#pragma unroll
    for (int c = 0; c < BC; ++c) {
        const int v = tid + c * NT;
        if constexpr (!BT) b_off[c] = (uint32_t)(((n0 + (v >> 3)) * g.ldb + kb + (v & 7) * 8) * 2);
        else b_off[c] = (uint32_t)((((int64_t)kb + v / BQ) * g.ldb + n0 + (v % BQ) * 8) * 2);
    }
    const uint32_t bt_row = (uint32_t)(g.ldb * 2);

    u32x4_v ra[AC], rb[BC];
    auto load_global = [&](int kt) {
        const int kofs = kt * BK;
#pragma unroll
        for (int c = 0; c < AC; ++c)
            ra[c] = __builtin_bit_cast(u32x4_v, __builtin_amdgcn_raw_buffer_load_b128(ar, a_off[c], kofs * 2, 0));
        const uint32_t s = BT ? (uint32_t)kofs * bt_row : (uint32_t)kofs * 2;
#pragma unroll
        for (int c = 0; c < BC; ++c)
            rb[c] = __builtin_bit_cast(u32x4_v, __builtin_amdgcn_raw_buffer_load_b128(br, b_off[c], s, 0));
    };
    auto store_lds = [&](int buf) {
        uint16_t *As = lds + buf * STAGE;
        uint16_t *Bs = As + BM * LDK;
#pragma unroll
        for (int c = 0; c < AC; ++c) {
            const int v = tid + c * NT;
            *(u32x4_v *)(As + (v >> 3) * LDK + (v & 7) * 8) = ra[c];
        }
#pragma unroll
        for (int c = 0; c < BC; ++c) {
            const int v = tid + c * NT;
            if constexpr (!BT) *(u32x4_v *)(Bs + (v >> 3) * LDK + (v & 7) * 8) = rb[c];
            else *(u32x4_v *)(Bs + (v / BQ) * LDN + (v % BQ) * 8) = rb[c];
        }
    };

    f32x16_t acc[2][TN];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // transpose-read addressing of the k-major B fragments (see above):
    // 16-lane group gi covers columns 16 (gi & 1).. and k rows 8 (gi >> 1)..
    const int gi = lane >> 4, si = lane & 15;
    static_assert(BM * (BN + 8) <= 2 * STAGE, "epilogue tile fits the stages");
    const int tr_off = (8 * (gi >> 1) + (si >> 2)) * LDN + 16 * (gi & 1) + 4 * (si & 3);
    auto compute = [&](int buf) {
        const uint16_t *As = lds + buf * STAGE;
        const uint16_t *Bs = As + BM * LDK;
        const int arow = wm * 64 + (lane & 31);
        const int brow = wn * (BN / 2) + (lane & 31);
        const int kof = 8 * (lane >> 5);
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            bf16x8_t a[2], b[TN];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = *(const bf16x8_t *)(As + (arow + i * 32) * LDK + s * 16 + kof);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (!BT) {
                    b[j] = *(const bf16x8_t *)(Bs + (brow + j * 32) * LDK + s * 16 + kof);
                } else {
                    const uint16_t *p = Bs + (s * 16) * LDN + wn * (BN / 2) + j * 32 + tr_off;
                    const v4s_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((IM_LDS3 v4s_t *)p);
                    const v4s_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((IM_LDS3 v4s_t *)(p + 4 * LDN));
                    const short v8[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    b[j] = __builtin_bit_cast(bf16x8_t, v8);
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };

    if (nk > 0) {
        load_global(0);
        store_lds(0);
        __syncthreads();
        if (nk > 1) load_global(1);
        for (int kt = 0; kt < nk; ++kt) {
            compute(kt & 1);
            if (kt + 1 < nk) store_lds((kt + 1) & 1);
            if (kt + 2 < nk) load_global(kt + 2);
            __syncthreads();
        }
    }

    // epilogue: lane (l & 31) holds sample column n, registers 4*grp + q the
    // rows 8*grp + 4*(l >> 5) + q of each 32 x 32 tile
    if constexpr (EPI == T_HIDDEN || EPI == T_MASK) {
        // bf16 tile staged in LDS as [m][n] (rows of BN + 8), then written in
        // 16-byte row pieces; the ReLU mask is read the same way
        constexpr int LDO = BN + 8;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int nl = wn * (BN / 2) + j * 32 + (lane & 31);
#pragma unroll
                for (int grp = 0; grp < 4; ++grp)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int ml = wm * 64 + i * 32 + 8 * grp + 4 * (lane >> 5) + q;
                        float v = acc[i][j][4 * grp + q];
                        if constexpr (EPI == T_HIDDEN) v = fmaxf(v + g.bias[m0 + ml], 0.0f);
                        lds[ml * LDO + nl] = f32_to_bf16_rne(v);
                    }
            }
        __syncthreads();
        // BM rows x BN/8 pieces of 8 samples
#pragma unroll
        for (int c = 0; c < BM * BQ / NT; ++c) {
            const int v = tid + c * NT;
            const int ml = v / BQ, pc = v % BQ;
            uint4 o = *(const uint4 *)(lds + ml * LDO + pc * 8);
            const int64_t off = (m0 + ml) * g.ldc + n0 + pc * 8;
            if constexpr (EPI == T_MASK) {
                uint32_t ow[4] = {o.x, o.y, o.z, o.w};
                const uint4 h = *(const uint4 *)(g.mask + (m0 + ml) * g.ldm + n0 + pc * 8);
                const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // keep each half where the activation (bf16) is > 0
                    const uint32_t lo = hw[k] & 0xFFFFu, hi = hw[k] >> 16;
                    const uint32_t keep = ((lo != 0 && !(lo & 0x8000u)) ? 0x0000FFFFu : 0u) |
                                          ((hi != 0 && !(hi & 0x8000u)) ? 0xFFFF0000u : 0u);
                    ow[k] &= keep;
                }
                o = make_uint4(ow[0], ow[1], ow[2], ow[3]);
                if (g.rs_part) {
                    // the row's sum over this tile's columns: the BQ consecutive lanes
                    // holding the row's pieces are summed by a fixed DPP pattern into
                    // the group's last lane
                    float rs = 0.0f;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        rs += bf16_to_f32((uint16_t)(ow[k] & 0xFFFFu)) + bf16_to_f32((uint16_t)(ow[k] >> 16));
                    rs = lane_group_sum<BQ>(rs);
                    if (pc == BQ - 1) g.rs_part[(m0 + ml) * (g.N / BN) + n0 / BN] = (double)rs;
                }
            }
            *(uint4 *)((uint16_t *)g.C + off) = o;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t n = n0 + wn * (BN / 2) + j * 32 + (lane & 31);
#pragma unroll
                for (int grp = 0; grp < 4; ++grp)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int64_t m = m0 + wm * 64 + i * 32 + 8 * grp + 4 * (lane >> 5) + q;
                        const float v = acc[i][j][4 * grp + q];
                        if constexpr (EPI == T_LINEAR) {
                            if (m < g.M_valid) ((float *)g.C)[m * g.ldc + n] = v + g.bias[m];
                        } else {
                            ((float *)g.C)[((int64_t)split * g.M + m) * g.ldc + n] = v;
                        }
                    }
            }
    }
}

// ---------------------------------------------------------------------------
// Forward and input-gradient products of the layers whose output width is a
// multiple of 256: C[256 m][128 n] tiles, the weights in MFMA fragment order
// (frag_index, K padded to 64), the k-major activations as in tgemm_kernel.
//
// What bounds tgemm_kernel on these shapes is LDS: a K step of a 256 x 256
// tile reads and writes 256 KB of it for 2048 cycles of MFMA.  Here the
// weight fragments come straight from the L2 into registers (1 KB of
// consecutive bytes per load, one K step ahead), so that only the activations
// pass through LDS (160 KB), and a block is 4 waves with 70 KB of LDS, two to
// a CU: one block's epilogue (the tile staged in LDS, then 64 KB of stores)
// runs beside the other's K loop.  A wave owns 64 rows x 128 columns (2 x 4
// MFMA tiles), the sums over k in the order of tgemm_kernel.
// Both networks' 1024 x 1024 layer over 524288 samples (2.2 TFLOP): 2.52 ms
// with tgemm_kernel, 2.04 here; their 1024 x 384 layer 1.7 -> 1.24 ms.  Of the
// 2.04, 1.39 are the K loop (25 GB of fragments and activations from the L2,
// at the 18 TB/s it delivers; the MFMA pipe is busy 59% of the kernel), the
// rest the outputs' 2.1 GB going to memory.  One block of 8 waves on 256
// columns (a third less L2 traffic, but no second block beside its epilogue)
// took 2.20 ms; starting every second block half a tile later, 2.1.
//
// K loop, step kt: LDS buffer kt & 1 holds the step's activations, rb (in
// flight) the next step's, wa the step's weight fragments.  The weight
// fragments of step kt + 1 are loaded right after the MFMAs that used their
// registers; rb is written to the other buffer after substep 0 (the buffer
// was last read before the previous step's barrier) and refilled with step
// kt + 2; the barrier after substep 2 lets substep 3 read the next step's
// first fragments ahead of its MFMAs.  Past the last step the loads go
// through descriptors of extent zero (no memory access).
// ---------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(256, 2) void fgemm_kernel(TGemmPair p)
{
    constexpr int BM = 256, BN = FGEMM_BN, BK = 64, NT = 256, TN = BN / 32, BQ = BN / 8;
    constexpr int LDN = BN + 32;      // LDS rows shifted by 64 bytes: the 4 rows x 64 bytes
                                      // a half wave's transpose read touches lie in distinct banks
    constexpr int STAGE = BK * LDN;
    constexpr int LDO = BN + 8;
    constexpr int LDS_ELEMS = BM * LDO > 2 * STAGE ? BM * LDO : 2 * STAGE;
    __shared__ __attribute__((aligned(16))) uint16_t lds[LDS_ELEMS];
    int id = xcd_order(blockIdx.x, gridDim.x);
    const bool second = id >= p.blocks0;
    if (second) id -= p.blocks0;
    const TGemm g = second ? p.g[1] : p.g[0];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mblocks = g.M / BM;
    const int64_t m0 = (int64_t)(id % mblocks) * BM;
    const int64_t n0 = (int64_t)(id / mblocks) * BN;
    const int nk = g.K / BK;
    uint4 mbits_in = make_uint4(0u, 0u, 0u, 0u);
    if constexpr (EPI == T_MASK) mbits_in = g.mbits[(int64_t)id * NT + tid];

    const __amdgpu_buffer_rsrc_t ar =
        __builtin_amdgcn_make_buffer_rsrc((void *)g.A, (short)0, (int)g.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t br =
        __builtin_amdgcn_make_buffer_rsrc((void *)g.B, (short)0, (int)g.b_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t none = __builtin_amdgcn_make_buffer_rsrc((void *)g.A, (short)0, 0, 0x00020000);

    // weight fragments: this lane's 16 bytes of a block, and the blocks of the
    // wave's two row tiles (4 KB per K step)
    const uint32_t a_vo = (uint32_t)(16 * lane);
    int a_so[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a_so[i] = ((int)(m0 / 32) + 2 * wave + i) * nk * 4096;
    // activations: 64 rows x 16 pieces of 8 samples, 4 per thread (16 rows apart)
    const uint32_t b_row = (uint32_t)(g.ldb * 2);
    const uint32_t b_vo = (uint32_t)(((int64_t)(tid / BQ) * g.ldb + n0 + (tid % BQ) * 8) * 2);
    u32x4_v wa[2][4], rb[4];
    auto load_a = [&](const __amdgpu_buffer_rsrc_t &r, int kt, int s) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            wa[i][s] = __builtin_bit_cast(u32x4_v, __builtin_amdgcn_raw_buffer_load_b128(
                                                       r, a_vo + 1024 * s, a_so[i] + kt * 4096, 0));
    };
    auto load_b = [&](const __amdgpu_buffer_rsrc_t &r, int kt) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            rb[c] = __builtin_bit_cast(u32x4_v, __builtin_amdgcn_raw_buffer_load_b128(
                                                    r, b_vo, (uint32_t)(kt * BK + 16 * c) * b_row, 0));
    };
    auto store_b = [&](int buf) {
        uint16_t *d = lds + buf * STAGE + (tid / BQ) * LDN + (tid % BQ) * 8;
#pragma unroll
        for (int c = 0; c < 4; ++c) *(u32x4_v *)(d + 16 * c * LDN) = rb[c];
    };
    // transpose read of the B fragments (as in tgemm_kernel)
    const int gi = lane >> 4, si = lane & 15;
    const int tr_off = (8 * (gi >> 1) + (si >> 2)) * LDN + 16 * (gi & 1) + 4 * (si & 3);
    bf16x8_t bn[TN];
    auto read_b = [&](int buf, int s) {
        const uint16_t *q = lds + buf * STAGE + s * 16 * LDN + tr_off;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const v4s_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((IM_LDS3 v4s_t *)(q + 32 * j));
            const v4s_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((IM_LDS3 v4s_t *)(q + 32 * j + 4 * LDN));
            const short v8[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            bn[j] = __builtin_bit_cast(bf16x8_t, v8);
        }
    };

    f32x16_t acc[2][TN];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    load_b(br, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) load_a(ar, 0, s);
    store_b(0);
    load_b(nk > 1 ? br : none, nk > 1 ? 1 : 0);
    __syncthreads();
    read_b(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        const bool more = kt + 1 < nk, more2 = kt + 2 < nk;
        const __amdgpu_buffer_rsrc_t an = more ? ar : none, bnx = more2 ? br : none;
        const int ka = more ? kt + 1 : 0, kb = more2 ? kt + 2 : 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            bf16x8_t b[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = bn[j];
            if (s == 3) {
                __syncthreads();
                read_b(buf ^ 1, 0);
            } else {
                read_b(buf, s + 1);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        b[j], __builtin_bit_cast(bf16x8_t, wa[i][s]), acc[i][j], 0, 0, 0);
            load_a(an, ka, s);
            if (s == 0) {
                store_b(buf ^ 1);
                load_b(bnx, kb);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();

    // epilogue: lane l holds row l & 31 of each 32 x 32 tile (the MFMA's first
    // operand is the activations), registers 4*grp + q the columns
    // 8*grp + 4*(l >> 5) + q; the half waves trade groups so that a lane holds
    // whole 16-byte pieces of its row; the tile is staged in LDS as [m][n],
    // then written in 16-byte pieces, 256 contiguous bytes per row
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int ml = wave * 64 + i * 32 + (lane & 31);
        float bias = 0.0f;
        if constexpr (EPI == T_HIDDEN) bias = g.bias[m0 + ml];
        uint16_t *row = lds + ml * LDO + 8 * (lane >> 5);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            uint32_t w[4][2];
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v[q] = acc[i][j][4 * grp + q];
                    if constexpr (EPI == T_HIDDEN) v[q] = fmaxf(v[q] + bias, 0.0f);
                }
                w[grp][0] = pack_bf16x2(v[0], v[1]);
                w[grp][1] = pack_bf16x2(v[2], v[3]);
            }
            const auto a0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
            const auto a1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
            const auto b0 = __builtin_amdgcn_permlane32_swap(w[2][0], w[3][0], false, false);
            const auto b1 = __builtin_amdgcn_permlane32_swap(w[2][1], w[3][1], false, false);
            *(u32x4_v *)(row + 32 * j) = u32x4_v{a0[0], a1[0], a0[1], a1[1]};
            *(u32x4_v *)(row + 32 * j + 16) = u32x4_v{b0[0], b1[0], b0[1], b1[1]};
        }
    }
    __syncthreads();
    // 16 pieces per thread; mask bits: word c / 4, bit 4 (c % 4) + k for the
    // low half of the piece's word k, 16 above it for the high half
    uint32_t mbits_out[4] = {0u, 0u, 0u, 0u};
    const uint32_t mbits_w[4] = {mbits_in.x, mbits_in.y, mbits_in.z, mbits_in.w};
#pragma unroll
    for (int c = 0; c < BM * BQ / NT; ++c) {
        const int ml = tid / BQ + c * (NT / BQ), pc = tid % BQ;
        const uint4 o = *(const uint4 *)(lds + ml * LDO + pc * 8);
        uint32_t ow[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int at = 4 * (c & 3) + k;
            if constexpr (EPI == T_HIDDEN) {
                // outputs are >= 0: bit 15 of each half becomes (half != 0)
                const uint32_t nz = ow[k] + 0x7FFF7FFFu;
                mbits_out[c >> 2] |= (nz >> (15 - at)) & (0x00010001u << at);
            } else {
                const uint32_t m = (mbits_w[c >> 2] >> at) & 0x00010001u;
                ow[k] &= (m << 16) - m;      // 0xFFFF in each half whose bit is set
            }
        }
        if constexpr (EPI == T_MASK) {
            // the row's sum over this tile's columns, from the 16 consecutive
            // lanes holding its pieces
            float rs = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                rs += __uint_as_float(ow[k] << 16) + __uint_as_float(ow[k] & 0xFFFF0000u);
            rs = lane_group_sum<BQ>(rs);
            if (pc == BQ - 1) g.rs_part[(m0 + ml) * (g.N / BN) + n0 / BN] = (double)rs;
        }
        *(uint4 *)((uint16_t *)g.C + (m0 + ml) * g.ldc + n0 + pc * 8) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
    }
    if constexpr (EPI == T_HIDDEN)
        g.mbits[(int64_t)id * NT + tid] = make_uint4(mbits_out[0], mbits_out[1], mbits_out[2], mbits_out[3]);
}

// ---------------------------------------------------------------------------
// Minibatch gather.  Column j = 64 c + l of the minibatch is env e0 + l of
// step t, where chunk c of the minibatch is q = perm[c]: t = q / (N/64),
// e0 = 64 (q % (N/64)).  One wavefront per chunk and part (blockIdx.y): parts
// of GATHER_ROWS observation rows, then parts of GATHER_COLS columns of the
// actions and of the means; chunks past the minibatch's end write zeros
// (padding columns).  One wavefront per chunk for everything left a small
// minibatch on 512 wavefronts (32768 samples of 226 rows: 38 us; by parts
// 17 us).  The chunk's actions and means ([64][A] floats, contiguous
// in the [T][N][A] storage) are read with loads of whole 128-byte row pieces
// into the wave's LDS slice (rows of 33 floats: the transposed reads hit 64
// distinct banks) and written out as [A][Mb] rows of 64 samples.
// ---------------------------------------------------------------------------
constexpr int GATHER_ROWS = 64, GATHER_COLS = 32;

__global__ __launch_bounds__(256) void gather_kernel(GatherArgs a)
{
    constexpr int KC = GATHER_COLS, LDC = KC + 1;
    __shared__ float gather_lds[4][64 * LDC];
    const int lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
    float *sh = gather_lds[threadIdx.x >> 6];
    if (c >= a.chunks_pad) return;
    const int64_t j = (int64_t)c * 64 + lane;
    const int64_t Mb = a.Mb_pad;
    const bool pad = c >= a.chunks;
    int q = pad ? 0 : a.perm[c];
    q = q < 0 ? 0 : (q >= a.n_chunks ? a.n_chunks - 1 : q);   // memory safety only
    const int64_t t = q / a.cpt;
    const int64_t e = (int64_t)(q % a.cpt) * 64 + lane;
    const int obs_parts = (a.K0 + GATHER_ROWS - 1) / GATHER_ROWS;
    int part = blockIdx.y;
    if (part < obs_parts) {
        int i = part * GATHER_ROWS;
        const int end = i + GATHER_ROWS < a.K0 ? i + GATHER_ROWS : a.K0;
        const int live = pad ? i : (end < a.D ? end : a.D);
        const float *o = a.obs + t * a.D * a.ld + e;
        for (; i + 16 <= live; i += 16) {
            float v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = o[(int64_t)(i + k) * a.ld];
#pragma unroll
            for (int k = 0; k < 16; ++k) a.x0[(i + k) * Mb + j] = f32_to_bf16_rne(v[k]);
        }
        for (; i < live; ++i) a.x0[i * Mb + j] = f32_to_bf16_rne(o[(int64_t)i * a.ld]);
        for (; i < end; ++i) a.x0[i * Mb + j] = 0;
        if (part == 0) {
            const int64_t s = t * a.ld + e;
            a.logp_old[j] = pad ? 0.0f : a.logp[s];
            a.adv[j] = pad ? 0.0f : a.adv_src[s];
            a.ret[j] = pad ? 0.0f : a.ret_src[s];
            a.vold[j] = pad ? 0.0f : a.value[s];
        }
        return;
    }
    part -= obs_parts;
    const int col_parts = (a.A + KC - 1) / KC;
    const bool means = part >= col_parts;
    const int k0 = (means ? part - col_parts : part) * KC;
    const int kc = a.A - k0 < KC ? a.A - k0 : KC;
    float *dst = (means ? a.mean_old : a.act) + k0 * Mb + j;
    if (pad) {
        for (int cc = 0; cc < kc; ++cc) dst[cc * Mb] = 0.0f;
        return;
    }
    const float *src = (means ? a.mean : a.action) + (t * a.N + (e - lane)) * a.A + k0;
    // the LDS slice is the wave's own and a wave's LDS operations complete
    // in order: no barrier between these writes and the reads below
#pragma unroll 16
    for (int x = lane; x < 64 * KC; x += 64) {
        const int r = x / KC, cc = x % KC;
        if (cc < kc) sh[r * LDC + cc] = src[(int64_t)r * a.A + cc];
    }
    for (int cc = 0; cc < kc; ++cc) dst[cc * Mb] = sh[lane * LDC + cc];
}

// ---------------------------------------------------------------------------
// Critic head (width-1 output layer) on feature-major activations.
// ---------------------------------------------------------------------------
// SPT samples per thread, a wavefront per block, each sample's sum over the rows
// in order; rows in chunks of 64 / SPT, two chunk buffers in turn, so that one to
// two chunks are in flight (rows past the last load the last).  Few samples want
// two each, so that more wavefronts share them (32768 samples of 512 rows: 23 us,
// with four 26), many want four, for longer reads (131072 samples 33 and 30 us,
// 524288 130 and 117; eight 172).
template <int SPT>
__global__ __launch_bounds__(64) void head_forward_kernel(const uint16_t *__restrict__ h, int K,
                                                          int64_t Mb, const float *__restrict__ w,
                                                          const float *__restrict__ b,
                                                          float *__restrict__ v)
{
    constexpr int C = 64 / SPT, W = SPT / 2;
    typedef uint32_t words_t __attribute__((ext_vector_type(W)));
    const int64_t j = ((int64_t)blockIdx.x * 64 + threadIdx.x) * SPT;
    words_t xa[C], xb[C];
    float wa, wb;      // the chunk's weights, one per lane
    auto load = [&](int k0, words_t (&x)[C], float &wl) {
        const int kw = k0 + (threadIdx.x & (C - 1));
        wl = w[kw < K ? kw : K - 1];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int k = k0 + i < K ? k0 + i : K - 1;
            x[i] = *(const words_t *)(h + k * Mb + j);
        }
    };
    float s[SPT];
#pragma unroll
    for (int q = 0; q < SPT; ++q) s[q] = 0.0f;
    auto sum = [&](int k0, const words_t (&x)[C], float wl) {
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (k0 + i >= K) break;
            const float wk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wl), i));
#pragma unroll
            for (int q = 0; q < W; ++q) {
                s[2 * q] += wk * __uint_as_float(x[i][q] << 16);
                s[2 * q + 1] += wk * __uint_as_float(x[i][q] & 0xFFFF0000u);
            }
        }
    };
    load(0, xa, wa);
    for (int k0 = 0; k0 < K; k0 += 2 * C) {
        load(k0 + C, xb, wb);
        sum(k0, xa, wa);
        load(k0 + 2 * C, xa, wa);
        if (k0 + C < K) sum(k0 + C, xb, wb);
    }
#pragma unroll
    for (int q = 0; q < SPT; q += 2) *(float2 *)(v + j + q) = make_float2(s[q] + b[0], s[q + 1] + b[0]);
}

// dZ^T[k][j] = w[k] dV[j] where h[k][j] > 0 (bf16), for the last hidden
// layer; rows K..gridDim.y-1 (padding) are zero.  8 samples per thread.
// Optionally the block's float64 partial sums of row k < K, at
// [k][blockIdx.x]: pw of h[k][j] dV[j] (the head's weight gradient), pb of
// the stored dZ^T[k][j] (the layer's bias gradient); each thread's 8 terms in
// order, a fixed wavefront butterfly, the 4 wave sums in wave order.
__global__ __launch_bounds__(256) void head_backward_kernel(const uint16_t *__restrict__ h, int K,
                                                            int64_t Mb,
                                                            const float *__restrict__ w,
                                                            const float *__restrict__ dv,
                                                            uint16_t *__restrict__ dz,
                                                            double *__restrict__ pw,
                                                            double *__restrict__ pb)
{
    __shared__ double red[2][4];
    const int64_t j = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    const int k = blockIdx.y;
    double sw = 0.0, sb = 0.0;
    if (j < Mb) {
        uint4 *out = (uint4 *)(dz + k * Mb + j);
        if (k >= K) {
            *out = make_uint4(0u, 0u, 0u, 0u);
        } else {
            const uint4 x = *(const uint4 *)(h + k * Mb + j);
            const float4 d0 = *(const float4 *)(dv + j), d1 = *(const float4 *)(dv + j + 4);
            const float d[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
            const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
            const float wk = w[k];
            uint32_t o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t lo = xw[q] & 0xFFFFu, hi = xw[q] >> 16;
                const uint32_t a = (lo != 0 && !(lo & 0x8000u)) ? f32_to_bf16_rne(wk * d[2 * q]) : 0u;
                const uint32_t b = (hi != 0 && !(hi & 0x8000u)) ? f32_to_bf16_rne(wk * d[2 * q + 1]) : 0u;
                o[q] = a | (b << 16);
                sw += (double)bf16_to_f32((uint16_t)lo) * (double)d[2 * q];
                sw += (double)bf16_to_f32((uint16_t)hi) * (double)d[2 * q + 1];
                sb += (double)bf16_to_f32((uint16_t)a);
                sb += (double)bf16_to_f32((uint16_t)b);
            }
            *out = make_uint4(o[0], o[1], o[2], o[3]);
        }
    }
    if (k >= K || (!pw && !pb)) return;     // uniform over the block
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sw += __shfl_xor(sw, o);
        sb += __shfl_xor(sb, o);
    }
    if (lane == 0) {
        red[0][wave] = sw;
        red[1][wave] = sb;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double t = ((red[threadIdx.x][0] + red[threadIdx.x][1]) + red[threadIdx.x][2]) +
                         red[threadIdx.x][3];
        double *p = threadIdx.x == 0 ? pw : pb;
        if (p) p[(int64_t)k * gridDim.x + blockIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// Sums of split partials (ReduceArgs): a weight block takes 256 outputs, one
// per thread, their splits added in order, 32 loads in flight at a time (one
// after the other, the 256 splits of a 28 x 512 layer took 31 us); a row
// block takes 4 rows, one per wavefront, the lanes every 64th partial, a
// fixed pattern over the lanes.  Bound by the partials' bytes
// (67 MB of 32 splits of two 512 x 1024 layers: 24 us).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void reduce_kernel(ReduceArgs r)
{
    constexpr int ZC = 32;
    int job = 0;
    bool rows = false;
    int b = blockIdx.x;
#pragma unroll
    for (int k = 2 * MAX_REDUCE - 1; k >= 0; --k)
        if (k < 2 * r.n && (int)blockIdx.x < r.end[k]) {
            job = k >> 1;
            rows = k & 1;
            b = (int)blockIdx.x - (k > 0 ? r.end[k - 1] : 0);
        }
    const ReduceJob g = job == 0 ? r.j[0] : (job == 1 ? r.j[1] : r.j[2]);
    const int tid = threadIdx.x;
    if (rows) {
        const int row = b * 4 + (tid >> 6), lane = tid & 63;
        if (row >= g.prows) return;
        double s = 0.0;
        const double *q = g.part + (int64_t)row * g.parts;
        if (g.pairs)
            for (int k = lane; k < g.parts / 2; k += 64) s += (double)((float)q[2 * k + 1] + (float)q[2 * k]);
        else
            for (int k = lane; k < g.parts; k += 64) s += q[k];
        s = wave_sum63(s);
        if (lane == 63) g.row_out[row] = (float)s;
        return;
    }
    const int idx = b * 256 + tid;
    if (idx >= g.rows * g.cols) return;
    const float *p = g.P + (int64_t)(idx / g.cols) * g.N + idx % g.cols;
    const int64_t stride = (int64_t)g.M * g.N;
    float s = 0.0f;
    int z = 0;
    for (; z + ZC <= g.S; z += ZC) {
        float x[ZC];
#pragma unroll
        for (int i = 0; i < ZC; ++i) x[i] = p[(z + i) * stride];
#pragma unroll
        for (int i = 0; i < ZC; ++i) s += x[i];
    }
#pragma unroll 8
    for (; z < g.S; ++z) s += p[z * stride];
    g.out[idx] = s;
}

// ---------------------------------------------------------------------------
// Loss: per sample, the clipped surrogate, value loss and KL; writes the
// bf16 output-layer gradient dmu^T [A][Mb] (zero for padding columns), dV,
// and per-block float64 partials of the loss fields, field-major.  A block
// takes 256 samples with four threads each, which split the actions (256
// consecutive threads read a 1 KB row piece): the terms of the
// log-likelihood and the KL pass through LDS by chunks of 16 actions, where
// one thread per sample each adds them in action order; then every wave sums
// its actions' partials over its lanes by a fixed pattern, the block's four
// waves of an action in order.  One thread per sample over all actions left
// 32768 samples on 128 blocks of 4 waves (28 actions: 43 us; 524288 samples
// of 69 actions 222 us; now 17 and 223 us, with the output layers' bias sums,
// 9 and 21 us as passes of their own).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void loss_kernel(LossArgs a)
{
    constexpr int KC = 16;
    __shared__ float sh_logp[2][KC][LOSS_BLOCK], sh_kl[2][KC][LOSS_BLOCK];
    __shared__ float sum_logp[LOSS_BLOCK];
    __shared__ double red[4][loss_fields(MAX_ACTIONS)];
    const int lane = threadIdx.x & 63, sj = threadIdx.x & (LOSS_BLOCK - 1);
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);     // actions grp, grp + 4, ...
    const int quarter = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
    const int64_t j = (int64_t)blockIdx.x * LOSS_BLOCK + sj;
    const int64_t Mb = a.Mb_pad;
    const bool live = j < a.Mb;
    float logp = 0.0f, kl = 0.0f;
    // two LDS buffers in turn: a chunk is overwritten two barriers after it was read
    for (int k0 = 0, p = 0; k0 < a.A; k0 += KC, p ^= 1) {
#pragma unroll
        for (int i = 0; i < KC / 4; ++i) {
            const int q = grp + 4 * i, k = k0 + q;
            if (k < a.A) {
                const float ls = a.log_std[k], lso = a.log_std_old[k];
                const float sig = expf(ls);
                const float sig2 = expf(2.0f * ls), so2 = expf(2.0f * lso);
                const float mu = a.mean[k * Mb + j];
                const float d = a.act[k * Mb + j] - mu;
                const float dm = a.mean_old[k * Mb + j] - mu;
                sh_logp[p][q][sj] = d * d / (2.0f * sig * sig) + ls + 0.91893853320467274f;
                sh_kl[p][q][sj] = ls - lso + (so2 + dm * dm) / (2.0f * sig2) - 0.5f;
            }
        }
        __syncthreads();
        const int n = a.A - k0 < KC ? a.A - k0 : KC;
        if (grp == 0) {
            for (int q = 0; q < n; ++q) logp -= sh_logp[p][q][sj];
        } else if (grp == 2) {
            for (int q = 0; q < n; ++q) kl += sh_kl[p][q][sj];
        }
    }
    if (grp == 0) sum_logp[sj] = logp;
    if (!live) kl = 0.0f;
    __syncthreads();
    logp = sum_logp[sj];
    const double n = (double)a.n_samples;
    const double amean = a.summary[IM_SUM_ADVANTAGE] / n;
    const double avar = (a.summary[IM_SUM_ADVANTAGE_SQ] - a.summary[IM_SUM_ADVANTAGE] * amean) / (n - 1.0);
    const double astd = sqrt(avar > 0.0 ? avar : 0.0);
    const float inv_mb = 1.0f / (float)a.Mb;
    float g_logp = 0.0f, l_pi = 0.0f, l_v = 0.0f, clipped = 0.0f, g_v = 0.0f;
    if (live) {
        const float ratio = expf(logp - a.logp_old[j]);
        const float A = (float)(((double)a.adv[j] - amean) / (astd + 1e-8));
        const float rc = fminf(fmaxf(ratio, 1.0f - a.clip), 1.0f + a.clip);
        const float s1 = -A * ratio, s2 = -A * rc;
        l_pi = fmaxf(s1, s2);
        g_logp = (s1 >= s2 ? -A * ratio : 0.0f) * inv_mb;
        clipped = fabsf(ratio - 1.0f) > a.clip ? 1.0f : 0.0f;
        // value loss
        const float V = a.value[j], R = a.ret[j], Vo = a.vold[j];
        float dv;
        if (a.clipped_value_loss) {
            const float dvo = V - Vo;
            const float Vc = Vo + fminf(fmaxf(dvo, -a.clip), a.clip);
            const float e1 = (V - R) * (V - R), e2 = (Vc - R) * (Vc - R);
            l_v = fmaxf(e1, e2);
            const bool inside = dvo > -a.clip && dvo < a.clip;
            dv = e1 >= e2 ? 2.0f * (V - R) : (inside ? 2.0f * (Vc - R) : 0.0f);
        } else {
            l_v = (V - R) * (V - R);
            dv = 2.0f * (V - R);
        }
        g_v = a.value_coef * dv * inv_mb;
    }
    auto put = [&](int f, double x) {
        x = wave_sum63(x);
        if (lane == 63) red[quarter][f] = x;
    };
    // per action: the mean's gradient (bf16), its sum (the bias gradient) and
    // the log-std gradient
#pragma unroll 2
    for (int k = grp; k < a.A; k += 4) {
        float gm = 0.0f;
        double x = 0.0;
        if (live) {
            const float sig2 = expf(2.0f * a.log_std[k]);
            const float d = a.act[k * Mb + j] - a.mean[k * Mb + j];
            gm = g_logp * d / sig2;
            x = (double)g_logp * ((double)d * d / sig2 - 1.0);
        }
        const uint16_t h = f32_to_bf16_rne(gm);
        a.dmu[k * Mb + j] = h;
        put(k, x);
        put(a.A + k, (double)bf16_to_f32(h));
    }
    if (grp == 0) {
        a.dv[j] = g_v;
        put(2 * a.A, (double)g_v);
        put(2 * a.A + 1, (double)l_pi);
    } else if (grp == 1) {
        put(2 * a.A + 2, (double)l_v);
    } else if (grp == 2) {
        put(2 * a.A + 3, (double)kl);
    } else {
        put(2 * a.A + 4, (double)clipped);
    }
    __syncthreads();
    const int nf = loss_fields(a.A);
    if ((int)threadIdx.x < nf) {
        const int f = threadIdx.x;
        a.partial[(int64_t)f * gridDim.x + blockIdx.x] = ((red[0][f] + red[1][f]) + red[2][f]) + red[3][f];
    }
}

// ---------------------------------------------------------------------------
// Optimizer.  norm_kernel: per-block float64 sums of g^2 over the flat
// gradient.  finalize_kernel (one block): the minibatch's log-std gradient
// (loss partials + entropy term) into the flat gradient, the loss stats,
// the global norm and clip factor, the KL-adaptive learning rate, the Adam
// step count and bias corrections.  adam_kernel: the step.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void norm_kernel(const float *__restrict__ g, int64_t P,
                                                   double *__restrict__ partial)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < P; i += (int64_t)gridDim.x * 256)
        s += (double)g[i] * (double)g[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// the log-std, output-bias gradients and loss stats of the minibatch from the
// loss partials: one block per field, a fixed tree over the blocks' partials
__global__ __launch_bounds__(256) void loss_reduce_kernel(LossReduceArgs r)
{
    __shared__ double red[256];
    const int f = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < r.blocks; b += 256) s += r.partial[(int64_t)f * r.blocks + b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    s = red[0];
    const int A = r.A;
    if (f < A) r.grad_log_std[f] = (float)(s - (double)r.entropy_coef);
    else if (f < 2 * A) r.grad_bias[f - A] = (float)s;
    else if (f == 2 * A) *r.grad_vbias = (float)s;
    else r.mb_stats[f - 2 * A - 1] = s / (double)r.Mb;
}

__global__ __launch_bounds__(256) void finalize_kernel(FinalizeArgs f)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int b = threadIdx.x; b < f.norm_blocks; b += 256) s += f.norm_partial[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double norm = sqrt(red[0]);
    double scale = 1.0;
    if (f.max_grad_norm > 0.0f) {
        const double coef = (double)f.max_grad_norm / (norm + 1e-6);
        if (coef < 1.0) scale = coef;
    }
    const double kl = f.mb_stats[2];
    float lr = *f.lr;
    if (f.desired_kl > 0.0f) {
        if (kl > 2.0 * f.desired_kl) lr = fmaxf(f.lr_min, lr / 1.5f);
        else if (kl > 0.0 && kl < 0.5 * f.desired_kl) lr = fminf(f.lr_max, lr * 1.5f);
    }
    *f.lr = lr;
    const int step = *f.step + 1;
    *f.step = step;
    f.opt->scale = (float)scale;
    f.opt->lr = lr;
    f.opt->bc1 = (float)(1.0 - pow((double)f.beta1, (double)step));
    f.opt->bc2 = (float)(1.0 - pow((double)f.beta2, (double)step));
    if (f.stats) {
        f.stats[IM_PPO_LOSS_PI] += f.mb_stats[0];
        f.stats[IM_PPO_LOSS_V] += f.mb_stats[1];
        f.stats[IM_PPO_KL] += f.mb_stats[2];
        f.stats[IM_PPO_CLIP_FRAC] += f.mb_stats[3];
        f.stats[IM_PPO_GRAD_NORM] += norm;
        f.stats[IM_PPO_MINIBATCHES] += 1.0;
        f.stats[IM_PPO_LR] = (double)lr;
    }
}

__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ x, float *__restrict__ m,
                                                   float *__restrict__ v,
                                                   const float *__restrict__ g, int64_t P,
                                                   const OptScalars *__restrict__ o, float beta1,
                                                   float beta2, float eps)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= P) return;
    const float gi = g[i] * o->scale;
    const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    x[i] -= o->lr * (mi / o->bc1) / (sqrtf(vi / o->bc2) + eps);
}

// ---------------------------------------------------------------------------
// Weight refresh from the float32 masters: the training copies W [Mp][Kp]
// and W^T [Kp][Mp] (bf16), and the rollout's packed copy [M_pad][K_pad]
// (roll_bf16 1: bf16; 2: float32 holding the bf16-rounded value; 0:
// float32) with its bias; padding stays zero.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void repack_kernel(RepackMulti p)
{
    int l = 0;
    while (l + 1 < p.n && (int)blockIdx.x >= p.end[l]) ++l;
    const RepackArgs &r = p.r[l];
    const int64_t idx = (int64_t)((int)blockIdx.x - (l ? p.end[l - 1] : 0)) * 256 + threadIdx.x;
    if (idx >= (int64_t)r.out * r.in) return;
    const int o = (int)(idx / r.in), i = (int)(idx % r.in);
    const float w = r.W[idx];
    const uint16_t h = f32_to_bf16_rne(w);
    if (r.wt) r.wt[r.wt_frag ? frag_index(o, i, r.Kp / 64) : (int64_t)o * r.Kp + i] = h;
    if (r.wtt) r.wtt[r.wtt_frag ? frag_index(i, o, r.Mp / 64) : (int64_t)i * r.Mp + o] = h;
    if (r.roll) {
        if (r.roll_bf16 == 1) ((uint16_t *)r.roll)[(int64_t)o * r.roll_K + i] = h;
        else if (r.roll_bf16 == 2) ((float *)r.roll)[(int64_t)o * r.roll_K + i] = bf16_to_f32(h);
        else ((float *)r.roll)[(int64_t)o * r.roll_K + i] = w;
    }
    if (r.rollf) r.rollf[frag_index(o, i, r.roll_K / 64)] = h;
    if (i == 0) {
        if (r.bias_train) r.bias_train[o] = r.b[o];
        if (r.bias_roll) r.bias_roll[o] = r.b[o];
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
hipError_t launch_tgemm(bool bt, int epi, TGemmPair p, hipStream_t s)
{
    const bool frag = fgemm_ok(epi, p.g[0].M);
    const bool bigm = tgemm_bm(p.g[0].M) == 256;
    const int bm = bigm ? 256 : 128, bn = frag ? FGEMM_BN : 256;
    int blocks[2] = {0, 0};
    for (int k = 0; k < p.n; ++k) {
        const TGemm &g = p.g[k];
        if (tgemm_bm(g.M) != bm || g.M % bm || g.N % 256 || g.K % 64) return hipErrorInvalidValue;
        if (frag && (!g.mbits || (epi == T_MASK && !g.rs_part))) return hipErrorInvalidValue;
        blocks[k] = (g.M / bm) * (g.N / bn) * p.splits[k];
    }
    p.blocks0 = blocks[0];
    const dim3 grid((unsigned)(blocks[0] + blocks[1]));
    if (frag && bt) {
        if (epi == T_HIDDEN) hipLaunchKernelGGL(fgemm_kernel<T_HIDDEN>, grid, dim3(256), 0, s, p);
        else hipLaunchKernelGGL(fgemm_kernel<T_MASK>, grid, dim3(256), 0, s, p);
    } else if (bt) {
        if (bigm) return hipErrorInvalidValue;
        if (epi == T_HIDDEN) hipLaunchKernelGGL((tgemm_kernel<true, T_HIDDEN, 2>), grid, dim3(256), 0, s, p);
        else if (epi == T_MASK) hipLaunchKernelGGL((tgemm_kernel<true, T_MASK, 2>), grid, dim3(256), 0, s, p);
        else if (epi == T_LINEAR) hipLaunchKernelGGL((tgemm_kernel<true, T_LINEAR, 2>), grid, dim3(256), 0, s, p);
        else return hipErrorInvalidValue;
    } else {
        if (epi != T_PARTIAL) return hipErrorInvalidValue;
        if (bigm) hipLaunchKernelGGL((tgemm_kernel<false, T_PARTIAL, 4>), grid, dim3(512), 0, s, p);
        else hipLaunchKernelGGL((tgemm_kernel<false, T_PARTIAL, 2>), grid, dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_gather(const GatherArgs &a, hipStream_t s)
{
    const int parts = (a.K0 + GATHER_ROWS - 1) / GATHER_ROWS + 2 * ((a.A + GATHER_COLS - 1) / GATHER_COLS);
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)((a.chunks_pad + 3) / 4), (unsigned)parts), dim3(256),
                       0, s, a);
    return hipGetLastError();
}

hipError_t launch_head_forward(const uint16_t *h, int K, int64_t Mb, const float *w, const float *b,
                               float *v, hipStream_t s)
{
    // Mb is a multiple of 256
    if (Mb >= 131072)
        hipLaunchKernelGGL(head_forward_kernel<4>, dim3((unsigned)(Mb / 256)), dim3(64), 0, s, h, K, Mb, w, b, v);
    else
        hipLaunchKernelGGL(head_forward_kernel<2>, dim3((unsigned)(Mb / 128)), dim3(64), 0, s, h, K, Mb, w, b, v);
    return hipGetLastError();
}

hipError_t launch_head_backward(const uint16_t *h, int K, int rows, int64_t Mb, const float *w,
                                const float *dv, uint16_t *dz, double *pw, double *pb, hipStream_t s)
{
    // Mb is a multiple of 256: 8 samples per thread
    hipLaunchKernelGGL(head_backward_kernel, dim3((unsigned)((Mb / 8 + 255) / 256), (unsigned)rows),
                       dim3(256), 0, s, h, K, Mb, w, dv, dz, pw, pb);
    return hipGetLastError();
}

hipError_t launch_reduce(ReduceArgs r, hipStream_t s)
{
    int end = 0;
    for (int k = 0; k < r.n; ++k) {
        const ReduceJob &g = r.j[k];
        end += (g.rows * g.cols + 255) / 256;
        r.end[2 * k] = end;
        end += (g.prows + 3) / 4;
        r.end[2 * k + 1] = end;
    }
    if (end == 0) return hipSuccess;
    hipLaunchKernelGGL(reduce_kernel, dim3((unsigned)end), dim3(256), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_loss(const LossArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(loss_kernel, dim3((unsigned)(a.Mb_pad / LOSS_BLOCK)), dim3(4 * LOSS_BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_loss_reduce(const LossReduceArgs &r, hipStream_t s)
{
    hipLaunchKernelGGL(loss_reduce_kernel, dim3((unsigned)loss_fields(r.A)), dim3(256), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_optimizer(const float *grad, int64_t P, double *norm_partial, int norm_blocks,
                            const FinalizeArgs &f, float *x, float *m, float *v, hipStream_t s)
{
    hipLaunchKernelGGL(norm_kernel, dim3((unsigned)norm_blocks), dim3(256), 0, s, grad, P, norm_partial);
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(256), 0, s, f);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, x, m, v, grad, P,
                       f.opt, f.beta1, f.beta2, f.eps);
    return hipGetLastError();
}

hipError_t launch_repack(RepackMulti r, hipStream_t s)
{
    int end = 0;
    for (int l = 0; l < r.n; ++l) {
        end += (int)(((int64_t)r.r[l].out * r.r[l].in + 255) / 256);
        r.end[l] = end;
    }
    if (end == 0) return hipSuccess;
    hipLaunchKernelGGL(repack_kernel, dim3((unsigned)end), dim3(256), 0, s, r);
    return hipGetLastError();
}

}  // namespace im
