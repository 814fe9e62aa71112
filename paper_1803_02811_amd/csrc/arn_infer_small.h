// Inference for small and middle batches, where latency is what counts: two launches for the policy/value and
// action-value heads (convolutions; fc layer + head + outputs), each spread over as many CUs as the batch allows.
//
//   infer_conv_band_kernel   one sample's last feature map is cut into bands of rows; a workgroup computes one band and
//                            recomputes the rows of the earlier layers that the band's windows reach into
//   fc_small_kernel          one workgroup per 16*NT hidden units and 16*MT samples (fc_small_tile), no k ranges in memory: the
//                            wavefronts of the workgroup share the contraction and add up through LDS.  With FC_HEAD it
//                            also multiplies its units into the head, 16 at a time; the last workgroup of a sample tile to
//                            finish adds the HIDN/16 contributions in order and writes the outputs
// Sums are formed in the same order for every batch size these kernels serve, so a sample's outputs do not depend on
// the batch it is in.
#pragma once
#include "arn_infer_fwd.h"
#include "arn_pv_head.h"

namespace arn {

// ---------------------------------------------------------------------------------------------------------------
// What bounds it: the latency of one sample's dependent layers.  At 16 samples and 84x84, a workgroup per sample leaves
// 240 CUs idle; with seven bands of one row (112 workgroups) a workgroup does 0.40 / 0.33 / 0.14 of the three layers.
// Inside a workgroup the first bound is what goes through the CU's 64 bytes per clock from the L2: with conv2 and conv3
// split over channel tiles and position tiles the eight wavefronts fetched 400 KB of weights, 5100 clocks before the
// first MFMA (cycle stamps).  Here every weight is fetched once per workgroup (twice in the 2-convolution network): conv1's
// go through LDS, conv2's and conv3's are split over channel tiles and halves of the contraction, and the two halves'
// sums meet in LDS.
struct BandPlan {
    int rows, bands;   // rows of the last feature map per workgroup, workgroups per sample
};
// as many bands as fit one workgroup per CU
template <class Geo>
inline BandPlan band_plan(int B) {
    BandPlan p{Geo::HL, 1};
    for (int rows = 1; rows <= Geo::HL; ++rows) {
        const int bands = (Geo::HL + rows - 1) / rows;
        if ((long)B * bands <= 256) { p.rows = rows; p.bands = bands; break; }
    }
    return p;
}

// Sample and band of block b of n: all bands of eight (at the end of the grid four, or one) consecutive samples on one XCD
// (see sample_block).
__device__ __forceinline__ void band_of_block(int b, int n, int bands, int &s, int &band) {
    const int chunk = b / (64 * bands), r = b - chunk * 64 * bands, left = n / bands - chunk * 64;
    const int run = left >= 64 ? 8 : left >= 32 && r < 32 * bands ? 4 : 1;
    if (run > 1) {
        s = chunk * 64 + (r & 7) * run + (r >> 3) % run;
        band = (r >> 3) / run;
    } else {
        s = b / bands;
        band = b - s * bands;
    }
}

// LDS of infer_conv_band_kernel: frame image (later the scratch of the half sums), act1 image, act2 image, conv1's weights
// (in the act2 image where that is large enough: they are dead before act2 is written)
template <class Geo, class P2, class P3>
struct BandLds {
    static constexpr int FRAME = 2 * Geo::OBS_BYTES, A1 = P2::IMG, A2 = Geo::HAS3 ? P3::IMG : 0, W1 = Geo::NC1 * KW1 * 2;
    static constexpr bool SHARE = A2 >= W1;
    static constexpr int A1_AT = FRAME, A2_AT = A1_AT + A1, W1_AT = SHARE ? A2_AT : A2_AT + A2;
    static constexpr int BIAS_AT = SHARE ? A2_AT + A2 : W1_AT + W1, BYTES = BIAS_AT + (Geo::NC1 + Geo::NC2 + (Geo::HAS3 ? C3 : 0)) * 4;
};

// One layer on one wavefront: channel tile fixed, position tiles first, first + step, ... of the n positions from p0 on, half
// of the k-steps (weights w).  The partner wavefront holds the other half; of their tiles the wavefront `half` finishes
// those with index parity `half` and hands the other sums to its partner through scratch.
template <class P, int KH, int MAXT, class Store>
__device__ __forceinline__ void band_layer(const char *img, const f16x8 (&w)[KH], int half, int p0, int n, int first, int step, int lane,
                                           f32x4 *own, f32x4 *partner, Store store) {
    const int li = lane & 15, lg = lane >> 4;
    const int nt = (n + 15) / 16, mine = (nt - first + step - 1) / step;   // this wavefront's tiles (uniform)
    auto base_of = [&](int i) __attribute__((always_inline)) {
        int row = (first + i * step) * 16 + li;
        row = row < n ? row : n - 1;
        return P::base_off(p0 + row) + P::lane_off(lg) + (half ? P::step_off(KH) : 0);
    };
    f32x4 keep[(MAXT + 1) / 2];
    f16x8 f[2][KH];
    auto load = [&](int i, f16x8 (&x)[KH]) __attribute__((always_inline)) {
        const int base = base_of(i);
#pragma unroll
        for (int j = 0; j < KH; ++j) {
            // step_off is not linear in the k-step: both halves' offsets are constants, chosen by the wavefront's half
            const int o = half ? P::step_off(KH + j) - P::step_off(KH) : P::step_off(j);
            x[j] = as_f16x8(*reinterpret_cast<const u32x4 *>(img + base + o));
        }
    };
    if (mine > 0) load(0, f[0]);
#pragma unroll
    for (int i = 0; i < MAXT; ++i) {
        if (i >= mine) break;
        if (i + 1 < mine) load(i + 1, f[(i + 1) & 1]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KH; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j], f[i & 1][j], acc, 0, 0, 0);
        if ((i & 1) == half) keep[i >> 1] = acc;
        else partner[(i >> 1) * 64 + lane] = acc;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MAXT; ++i) {
        if (i >= mine) break;
        if ((i & 1) != half) continue;
        const f32x4 o = own[(i >> 1) * 64 + lane], k = keep[i >> 1];
        const f32x4 v = half ? o + k : k + o;                    // first half + second half on both sides
        const int row = (first + i * step) * 16 + li;
        if (row < n) store(p0 + row, v);
    }
}

// eight uint8 (two little-endian words) -> eight fp16, exact: the bytes become the low mantissa bits of 1024 + b, and 1024
// is subtracted (a byte permute and one packed fp16 addition per
// pair instead of five instructions; its constants cost registers, which the kernels above do not have)
__device__ __forceinline__ u32x4 u8x8_to_f16x8_perm(uint32_t lo, uint32_t hi) {
    auto two = [](uint32_t v, uint32_t sel) -> uint32_t {
        const f16x2 h = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x64646464u, v, sel));
        const f16x2 k = {(_Float16)1024.f, (_Float16)1024.f};
        return __builtin_bit_cast(uint32_t, h - k);
    };
    // selector bytes: 0-3 = byte of v, 4-7 = a byte of 0x64646464
    u32x4 r;
    r.x = two(lo, 0x04010400u);
    r.y = two(lo, 0x04030402u);
    r.z = two(hi, 0x04010400u);
    r.w = two(hi, 0x04030402u);
    return r;
}

template <class Geo, class P2, class P3>
__global__ __launch_bounds__(INF_THREADS) void infer_conv_band_kernel(const InferConvArgs a, int rows, int bands) {
    constexpr int IN_H = Geo::IN_H, IN_W = Geo::IN_W, W1 = Geo::W1, W2 = Geo::W2, W3 = Geo::W3, OBS_BYTES = Geo::OBS_BYTES;
    constexpr int KS1 = KW1 / 32, KH2 = Geo::KW2 / 64, KH3 = KW3 / 64;
    constexpr bool HAS3 = Geo::HAS3;
    constexpr int W4 = 4 * IN_W / 16;                       // 16-byte words in four rows of a channel plane
    constexpr int NL = (4 * W4 * (Geo::H1 + 1) + INF_THREADS - 1) / INF_THREADS;
    constexpr int CT1 = Geo::NC1 / 16, CT2 = Geo::NC2 / 16, PG = 4 / CT2;   // channel tiles; position groups of conv2 / conv3
    constexpr int MAXT2 = ((Geo::P2 + 15) / 16 + PG - 1) / PG, MAXT3 = HAS3 ? (Geo::P3 + 15) / 16 : 1;
    constexpr int MAXT = MAXT2 > MAXT3 ? MAXT2 : MAXT3, SCR = (MAXT + 1) / 2 * 64;   // scratch words per wavefront
    typedef BandLds<Geo, P2, P3> L;
    static_assert((4 * IN_W) % 16 == 0 && layout_is_uniform<P2>() && layout_is_uniform<P3>(), "layouts");
    static_assert(L::BYTES <= 160 * 1024 && 8 * SCR * 16 <= L::FRAME && L::A1_AT % 16 == 0 && L::A2_AT % 16 == 0 && L::W1_AT % 16 == 0, "LDS budget");
    static_assert(PG >= 1 && (!HAS3 || PG == 1), "two halves of the contraction, CT2 channel tiles, PG position groups");
    constexpr int NW1 = L::W1 / 16 / INF_THREADS;
    static_assert(L::W1 / 16 % INF_THREADS == 0, "conv1's weights in whole words per thread");

    __shared__ u32x4 lds[L::BYTES / 16];
    u32x4 *const s_img = lds;                               // fp16 [4][IN_H][IN_W]; only the rows the band needs are filled
    char *const img = reinterpret_cast<char *>(lds);
    char *const a1l = img + L::A1_AT;
    char *const a2l = img + L::A2_AT;
    u32x4 *const s_w1 = reinterpret_cast<u32x4 *>(img + L::W1_AT);
    float *const s_bias = reinterpret_cast<float *>(img + L::BIAS_AT);
    f32x4 *const scratch = reinterpret_cast<f32x4 *>(lds);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    int s, band;
    band_of_block(blockIdx.x, gridDim.x, bands, s, band);
    typedef LastActs<Geo::NCL, Geo::PL> Out;   // fragment order: this kernel serves only batches of fc_small_kernel

    // rows of each layer's output that this band needs
    int r2_0, r2_1, r3_0 = 0, r3_1 = 0;
    if constexpr (HAS3) {
        r3_0 = band * rows;
        r3_1 = min(r3_0 + rows, Geo::H3);
        r2_0 = max(r3_0 - Geo::PAD3, 0);
        r2_1 = min(r3_1 - 1 - Geo::PAD3 + K3, Geo::H2);
    } else {
        r2_0 = band * rows;
        r2_1 = min(r2_0 + rows, Geo::H2);
    }
    const int r1_0 = max(S2 * r2_0 - Geo::PAD2, 0), r1_1 = min(S2 * (r2_1 - 1) - Geo::PAD2 + K2, Geo::H1);

    // the frame rows 4 r1_0 .. 4 (r1_1 - 1) + 7 of the four planes (words past the end repeat the last one)
    const int nw = W4 * (r1_1 - r1_0 + 1), w0 = W4 * r1_0;
    const u32x4 *src = reinterpret_cast<const u32x4 *>(a.obs + (size_t)s * OBS_BYTES);
    u32x4 rimg[NL];
    auto word = [&](int i) __attribute__((always_inline)) {
        int idx = tid + INF_THREADS * i;
        idx = idx < 4 * nw ? idx : 4 * nw - 1;
        const int ch = (idx >= nw) + (idx >= 2 * nw) + (idx >= 3 * nw);
        return ch * (IN_H * IN_W / 16) + w0 + idx - ch * nw;
    };
#pragma unroll
    for (int i = 0; i < NL; ++i)
        if (INF_THREADS * i < 4 * nw) rimg[i] = src[word(i)];
    // weights in the order they are needed
    u32x4 rw1[NW1];
#pragma unroll
    for (int i = 0; i < NW1; ++i) rw1[i] = reinterpret_cast<const u32x4 *>(a.w1)[tid + INF_THREADS * i];
    const int ct = wave % CT2, half = (wave / CT2) & 1, pg = wave / (2 * CT2);
    const int pair = wave ^ CT2;                             // the wavefront with the other half
    f16x8 w2[KH2], w3[HAS3 ? KH3 : 1];
#pragma unroll
    for (int j = 0; j < KH2; ++j)
        w2[j] = as_f16x8(*reinterpret_cast<const u32x4 *>(a.w2 + frag_base(ct, Geo::KW2, lane) + FRAG_STEP * (half * KH2 + j)));
    constexpr int NB = Geo::NC1 + Geo::NC2 + (HAS3 ? C3 : 0);
    float rb = 0.f;
    if (tid < NB) rb = tid < Geo::NC1 ? a.b1[tid] : tid < Geo::NC1 + Geo::NC2 ? a.b2[tid - Geo::NC1] : a.b3[tid - Geo::NC1 - Geo::NC2];
    __builtin_amdgcn_sched_barrier(0);
    clear_counters(a);
    if constexpr (P2::ZERO_FILL) {   // zero borders of the padded layers
        for (int i = tid; i < L::A1 / 16; i += INF_THREADS) lds[L::A1_AT / 16 + i] = zero_u4();
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        if (tid + INF_THREADS * i < 4 * nw) {
            const int at = 2 * word(i);
            s_img[at] = u8x8_to_f16x8_perm(rimg[i].x, rimg[i].y);
            s_img[at + 1] = u8x8_to_f16x8_perm(rimg[i].z, rimg[i].w);
        }
    }
#pragma unroll
    for (int i = 0; i < NW1; ++i) s_w1[tid + INF_THREADS * i] = rw1[i];
    if (tid < NB) s_bias[tid] = rb;
    __syncthreads();
    // conv3's weights are asked for only now: every load instruction takes 16 clocks of the CU's address unit, and the frame
    // is staged by wavefronts that have issued theirs
    if constexpr (HAS3) {
#pragma unroll
        for (int j = 0; j < KH3; ++j)
            w3[j] = as_f16x8(*reinterpret_cast<const u32x4 *>(a.w3 + frag_base(ct, KW3, lane) + FRAG_STEP * (half * KH3 + j)));
        __builtin_amdgcn_sched_barrier(0);
    }
    const float4 *const bias1 = reinterpret_cast<const float4 *>(s_bias + 4 * lg);
    const float4 *const bias2p = reinterpret_cast<const float4 *>(s_bias + Geo::NC1 + ct * 16 + 4 * lg);
    const float4 *const bias3p = reinterpret_cast<const float4 *>(s_bias + Geo::NC1 + Geo::NC2 + ct * 16 + 4 * lg);

    // ---- conv1: frame image -> act1 image; a wavefront takes all channels of every eighth position tile ----
    {
        f16x8 w1[CT1][KS1];
#pragma unroll
        for (int c = 0; c < CT1; ++c)
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) w1[c][ks] = as_f16x8(s_w1[(c * KS1 + ks) * 64 + lane]);
        const int p1_0 = r1_0 * W1, p1_1 = r1_1 * W1;
#pragma unroll 1
        for (int t = wave; p1_0 + t * 16 < p1_1; t += 8) {
            int pos = p1_0 + t * 16 + li;
            const bool valid = pos < p1_1;
            pos = valid ? pos : p1_1 - 1;
            const int oy = pos / W1, ox = pos - oy * W1;
            const int base = ((S1 * oy + lg) * IN_W + S1 * ox) * 2;
            u32x2 f[2 * KS1];
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) {
                const int off = base + ((ks >> 1) * (IN_H * IN_W) + (ks & 1) * 4 * IN_W) * 2;
                f[2 * ks] = *reinterpret_cast<const u32x2 *>(img + off);
                f[2 * ks + 1] = *reinterpret_cast<const u32x2 *>(img + off + 8);
            }
            f32x4 acc[CT1];
#pragma unroll
            for (int c = 0; c < CT1; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) {
                const f16x8 b = as_f16x8(u32x4{f[2 * ks].x, f[2 * ks].y, f[2 * ks + 1].x, f[2 * ks + 1].y});
#pragma unroll
                for (int c = 0; c < CT1; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[c][ks], b, acc[c], 0, 0, 0);
            }
            constexpr float sc = 1.0f / 255.0f;
            if (valid)
#pragma unroll
                for (int c = 0; c < CT1; ++c) {
                    const float4 b = bias1[4 * c];
                    *reinterpret_cast<u32x2 *>(a1l + P2::dst_off(pos) + (c * 16 + 4 * lg) * 2) =
                        relu_f16x4(acc[c][0] * sc + b.x, acc[c][1] * sc + b.y, acc[c][2] * sc + b.z, acc[c][3] * sc + b.w);
                }
        }
    }
    __syncthreads();
    if constexpr (HAS3 && P3::ZERO_FILL) {   // conv1's weights, which may share this image, are dead
        for (int i = tid; i < L::A2 / 16; i += INF_THREADS) lds[L::A2_AT / 16 + i] = zero_u4();
    }
    // ---- conv2: act1 image -> act2 image, or the result ----
    band_layer<P2, KH2, MAXT2>(a1l, w2, half, r2_0 * W2, (r2_1 - r2_0) * W2, pg, PG, lane, scratch + wave * SCR, scratch + pair * SCR,
                               [&](int row, f32x4 v) __attribute__((always_inline)) {
        const float4 bias2 = *bias2p;
        const u32x2 r = relu_f16x4(v[0] + bias2.x, v[1] + bias2.y, v[2] + bias2.z, v[3] + bias2.w);
        if constexpr (HAS3) *reinterpret_cast<u32x2 *>(a2l + P3::dst_off(row) + (ct * 16 + 4 * lg) * 2) = r;
        else *reinterpret_cast<u32x2 *>(a.a3 + Out::template at<true>(s, row, ct * 16 + 4 * lg)) = r;
    });
    // ---- conv3: act2 image -> act3 in global memory ----
    if constexpr (HAS3) {
        __syncthreads();
        band_layer<P3, KH3, MAXT3>(a2l, w3, half, r3_0 * W3, (r3_1 - r3_0) * W3, 0, 1, lane, scratch + wave * SCR, scratch + pair * SCR,
                                   [&](int row, f32x4 v) __attribute__((always_inline)) {
            const float4 bias3 = *bias3p;
            *reinterpret_cast<u32x2 *>(a.a3 + Out::template at<true>(s, row, ct * 16 + 4 * lg)) =
                relu_f16x4(v[0] + bias3.x, v[1] + bias3.y, v[2] + bias3.z, v[3] + bias3.w);
        });
    }
}

// ---------------------------------------------------------------------------------------------------------------
// fc layer for small batches.  What bounds it: the operands' way from the L2 into the CUs and the latency of each
// dependent step.  Weights and activations are in fragment order, so every load is one contiguous kilobyte straight into
// an MFMA operand, several k-steps of them in flight; nothing is staged, and the wavefronts' shares of the contraction
// are added through LDS, so no fp32 partial sums go through memory.  Measured at 256 samples and 3136 inputs, one fp16
// product, back to back: 4.6 us with 32 x 32 outputs per workgroup (8.4 with the activations read from rows: a 64-byte
// piece of sixteen rows per load thrashes the L1; the LDS-staged GEMM in eight k ranges takes 8.4 plus the addition of its
// partial sums).
enum { FC_PARTIAL = 0,   // fp32 [B][HID] sums without bias (pv_head_kernel finishes the layer: one "k range")
       FC_HIDDEN = 1,    // h = relu(sum + bias) as bf16 hi / lo rows
       FC_HEAD = 2 };    // h stays on chip: head, outputs
struct FcSmallArgs {
    const void *act;           // fp16 activations, or their bf16 hi part: fragment order over (sample, input)
    const __bf16 *act_lo;
    const void *w;             // fp16 (bf16 hi) weights in fragment order
    const __bf16 *w_lo;
    int B;
    float *partial;            // FC_PARTIAL
    const float *bias;
    __bf16 *h, *h_lo;          // FC_HIDDEN
    PvHeadArgs head;           // FC_HEAD: weights, bias and outputs
    float *zp;                 // FC_HEAD: [HID/16][samples padded to the tile][32] contributions to the head outputs
    unsigned *counters;        // FC_HEAD: one per sample tile, zero at launch
};

// wavefronts and k-steps per wavefront of a contraction over FEAT
template <int FEAT>
struct FcSmallSplit;
template <> struct FcSmallSplit<3136> { static constexpr int WAVES = 7, STEPS = 14; };
template <> struct FcSmallSplit<6912> { static constexpr int WAVES = 8, STEPS = 27; };
template <> struct FcSmallSplit<3456> { static constexpr int WAVES = 9, STEPS = 12; };
// wavefronts launched: at least eight, which the outputs of 32 samples take; the rest only help there
template <int FEAT>
constexpr int fc_small_threads() { return 64 * (FcSmallSplit<FEAT>::WAVES > 8 ? FcSmallSplit<FEAT>::WAVES : 8); }

// Values that workgroups of one launch hand to each other: agent-scope relaxed accesses bypass the caches that are not
// coherent between the XCDs, so no cache has to be written back or invalidated as a whole (a release / acquire pair
// around plain accesses took 14.9 instead of 12.1 us in a 256-sample trial).
__device__ __forceinline__ void store_agent(float *p, float a, float b) {
    const u32x2 v = {__float_as_uint(a), __float_as_uint(b)};
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_agent(const float *p) {
    return __uint_as_float(__hip_atomic_load(reinterpret_cast<const unsigned *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// NT, MT: tiles of 16 hidden units and of 16 samples per workgroup.  F16: one fp16 product; otherwise three bf16 products.
template <int FEAT, int HIDN, int NT, int MT, bool F16, int MODE>
__global__ __launch_bounds__(fc_small_threads<FEAT>()) void fc_small_kernel(const FcSmallArgs a) {
    constexpr int W = FcSmallSplit<FEAT>::WAVES, STEPS = FcSmallSplit<FEAT>::STEPS, PARTS = F16 ? 1 : 2;
    static_assert(W * STEPS * 32 == FEAT && HIDN % (16 * NT) == 0, "the wavefronts cover the contraction");
    // k-steps of loads in flight: what about 112 registers hold
    constexpr int FIT = 28 / ((NT + MT) * PARTS), DEPTH = FIT < STEPS ? FIT : STEPS;
    constexpr int NS = 16 * MT, TILE4 = NT * NS * 4;            // samples per workgroup; 16-byte words of its output tile
    __shared__ float4 red[W * TILE4];                           // [wavefront][unit tile][sample][16 units]
    __shared__ __attribute__((aligned(16))) __bf16 sH[2][TILE4 * 4];   // h, hi and lo, [unit tile][sample][16 units]
    __shared__ int s_last;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int x = blockIdx.x, m0 = blockIdx.y * NS, ks0 = wave * STEPS;

    u32x4 fw[DEPTH][NT][PARTS], fa[DEPTH][MT][PARTS];
    const char *wp[NT][PARTS], *ap[MT][PARTS];                  // wavefront-uniform; each lane reads 16 lane bytes further on
    const uint32_t lane16 = lane * 16;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const size_t at = ((size_t)(x * NT + n) * FEAT * 16 + (size_t)ks0 * FRAG_STEP) * 2;
        wp[n][0] = reinterpret_cast<const char *>(a.w) + at;
        if constexpr (!F16) wp[n][1] = reinterpret_cast<const char *>(a.w_lo) + at;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {   // the rows of samples past the batch are allocated; what they hold is never stored
        const size_t at = ((size_t)(blockIdx.y * MT + t) * FEAT * 16 + (size_t)ks0 * FRAG_STEP) * 2;
        ap[t][0] = reinterpret_cast<const char *>(a.act) + at;
        if constexpr (!F16) ap[t][1] = reinterpret_cast<const char *>(a.act_lo) + at;
    }
    auto load = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) {
#pragma unroll
            for (int n = 0; n < NT; ++n) fw[i % DEPTH][n][p] = *reinterpret_cast<const u32x4 *>(wp[n][p] + i * (FRAG_STEP * 2) + lane16);
#pragma unroll
            for (int t = 0; t < MT; ++t) fa[i % DEPTH][t][p] = *reinterpret_cast<const u32x4 *>(ap[t][p] + i * (FRAG_STEP * 2) + lane16);
        }
    };
    const bool worker = FcSmallSplit<FEAT>::WAVES >= 8 || wave < W;
    if (worker) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) load(i);
    }
    // head contribution: wavefront u takes head rows 16 (u & 1) .., sample tile (u / 2) % MT, unit tile u / (2 MT)
    const int hr = wave & 1, ht = (wave >> 1) % MT, hn = wave / (2 * MT);
    static_assert(MODE != FC_HEAD || (2 * MT * NT <= 8 && NS * 16 <= 512), "one head tile per wavefront, 16 lanes per sample");
    u32x4 hw = zero_u4(), hwl = zero_u4();
    float4 fc_bias = {};
    if constexpr (MODE == FC_HEAD) {
        const size_t at = frag_base(hr, HIDN, lane) + FRAG_STEP * ((x * NT + (hn < NT ? hn : 0)) >> 1);
        hw = *reinterpret_cast<const u32x4 *>(a.head.wh + at);
        hwl = *reinterpret_cast<const u32x4 *>(a.head.whl + at);
    }
    const int q = tid & 3, qm = (tid >> 2) % NS, qn = tid / (4 * NS);   // this thread's four units of one sample, below
    if constexpr (MODE != FC_PARTIAL) fc_bias = *reinterpret_cast<const float4 *>(a.bias + (x * NT + (qn < NT ? qn : 0)) * 16 + 4 * q);
    __builtin_amdgcn_sched_barrier(0);   // all of these loads are issued before the first is waited for

    f32x4 acc[NT][MT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (worker) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int d = i % DEPTH;
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    if constexpr (!F16) {
                        acc[n][t] = mfma_16x16x32<false>(fw[d][n][1], fa[d][t][0], acc[n][t]);
                        acc[n][t] = mfma_16x16x32<false>(fw[d][n][0], fa[d][t][1], acc[n][t]);
                    }
                    acc[n][t] = mfma_16x16x32<F16>(fw[d][n][0], fa[d][t][0], acc[n][t]);
                }
            if (i + DEPTH < STEPS) {
                load(i + DEPTH);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int t = 0; t < MT; ++t)
                red[wave * TILE4 + (n * NS + t * 16 + li) * 4 + lg] = make_float4(acc[n][t][0], acc[n][t][1], acc[n][t][2], acc[n][t][3]);
    }
    __syncthreads();
    // four units of one sample per thread, the wavefronts' shares added in order
    static_assert(TILE4 <= 64 * 7, "one pass over the tile");
    if (tid < TILE4) {
        float4 v = red[tid];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            const float4 u = red[w * TILE4 + tid];
            v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
        }
        const bool live = m0 + qm < a.B;
        const size_t at = (size_t)(m0 + qm) * HIDN + (x * NT + qn) * 16 + 4 * q;
        if constexpr (MODE == FC_PARTIAL) {
            if (live) *reinterpret_cast<float4 *>(a.partial + at) = v;
        } else {
            const float r0 = fmaxf(v.x + fc_bias.x, 0.f), r1 = fmaxf(v.y + fc_bias.y, 0.f), r2 = fmaxf(v.z + fc_bias.z, 0.f),
                        r3 = fmaxf(v.w + fc_bias.w, 0.f);
            if constexpr (MODE == FC_HIDDEN) {
                if (live) store_bf16x4_split(a.h, a.h_lo, at, r0, r1, r2, r3);
            } else {
                store_bf16x4_split(sH[0], sH[1], (size_t)tid * 4, r0, r1, r2, r3);
            }
        }
    }
    if constexpr (MODE == FC_HEAD) {
        __syncthreads();
        // contribution of each 16 units to the 32 head rows: half a k-step, the other half is zero (so that the bits do
        // not depend on NT)
        const int Mpad = gridDim.y * NS;
        if (hn < NT) {
            const int xn = x * NT + hn, at = (hn * NS + ht * 16 + li) * 16 + (lg & 1) * 8;
            const bool mine = (lg >> 1) == (xn & 1);
            u32x4 hh = *reinterpret_cast<const u32x4 *>(&sH[0][at]), hl = *reinterpret_cast<const u32x4 *>(&sH[1][at]);
            hh = mine ? hh : zero_u4();
            hl = mine ? hl : zero_u4();
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
            z = mfma_16x16x32<false>(hwl, hh, z);
            z = mfma_16x16x32<false>(hw, hl, z);
            z = mfma_16x16x32<false>(hw, hh, z);
            float *dst = a.zp + ((size_t)xn * Mpad + m0 + ht * 16 + li) * 32 + 16 * hr + 4 * lg;
            store_agent(dst, z[0], z[1]);
            store_agent(dst + 2, z[2], z[3]);
        }
        // The workgroup that finishes a sample tile last adds the contributions up.  Each wavefront waits for its stores
        // before the barrier, so the count that a workgroup adds follows all of them.
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        if (tid == 0)
            s_last = __hip_atomic_fetch_add(a.counters + blockIdx.y, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        __syncthreads();
        if (!s_last) return;
        const int c = tid & 15, m = tid >> 4, n = m0 + m;
        if (wave * 4 >= NS) return;              // whole wavefronts; 16 lanes per sample
        constexpr int NX = HIDN / 16;
        const bool live = n < a.B;
        const float *src = a.zp + (size_t)(m0 + m) * 32 + c;
        const float b0 = a.head.bh[c], b1 = a.head.bh[c + 16];
        float v0[NX], v1[NX];
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            v0[i] = load_agent(src + (size_t)i * Mpad * 32);
            v1[i] = load_agent(src + (size_t)i * Mpad * 32 + 16);
        }
        float z0 = 0.f, z1 = 0.f;
#pragma unroll
        for (int i = 0; i < NX; ++i) { z0 += v0[i]; z1 += v1[i]; }
        infer_outputs(a.head, n, live, c, z0 + b0, z1 + b1);
    }
}

}  // namespace arn
