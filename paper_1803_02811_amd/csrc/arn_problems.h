// The dense layers of the Nature CNN (fc and heads) written as instances of the two
// contraction kernels in arn_gemm.h: how each one gathers its activation operand,
// where its packed weights live and what its epilogue does.  (The convolutions have
// their own sample-resident kernels in arn_resident_conv.h / arn_resident.h.)
//
// Activations are NHWC bf16: act1 [B,20,20,32], act2 [B,9,9,64], act3 [B,7,7,64]
// (= the fc input with index (y*7+x)*64 + c; the packed fc weights are permuted
// to match), h [B,512]; with the 104x80 geometry [B,25,19,32], [B,12,9,64], [B,12,9,64].
// Gradients at pre-activations use the same layouts.  The fc problems are templates on
// the fc input size (3136 or 6912).
#pragma once
#include "arn_gemm.h"
#include "arn_layout.h"

namespace arn {

// fc: h = relu(act3 Wfc^T + b).  PARTIAL: each blockIdx.z covers a range of the contraction and writes an fp32
// partial [z][M][HIDN] (the only one, too, where pv_head_kernel finishes the layer); fc_finish_kernel or pv_head_kernel adds the
// partials in z order and applies bias, ReLU and the hi/lo split.  Otherwise ksplit is 1 and the epilogue does that directly.
template <int FEAT_, int HIDN, int BM_, bool PARTIAL>
struct FcFwdT {
    static constexpr int BM = BM_, RING = 2, K = FEAT_;
    static constexpr bool SHORT_K = false, WIDE = false, STORES_16BIT = !PARTIAL;
    static constexpr int PREFETCH_LOADS = 0;
    const __bf16 *in, *in_lo;
    int M;
    int ksplit;
    const __bf16 *w, *w_lo;
    const float *bias;
    __bf16 *out, *out_lo;
    float *partial;
    __device__ __forceinline__ const __bf16 *act() const { return in; }
    __device__ __forceinline__ const __bf16 *act_lo() const { return in_lo; }
    __device__ __forceinline__ const __bf16 *weights() const { return w; }
    __device__ __forceinline__ const __bf16 *weights_lo() const { return w_lo; }
    __device__ __forceinline__ int tiles() const { return HIDN / 16; }
    __device__ __forceinline__ float4 prefetch(int, int n) const { return *reinterpret_cast<const float4 *>(bias + n); }
    __device__ __forceinline__ void store(int m, int n, f32x4 v, int z, float4 b) const {
        if (m >= M) return;
        if constexpr (PARTIAL) {
            // the bias is read here too, so that it is in the L2s when the consumer adds it: without, pv_head_kernel waits for it from
            // memory (104x80, 512 samples: 6.7 instead of 5.8 us, in the gradient step of 2048 samples of 84x84 11.7 instead of 10.8)
            asm volatile("" ::"v"(b.x));
            *reinterpret_cast<float4 *>(partial + ((size_t)z * M + m) * HIDN + n) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
            store_bf16x4_split(out, out_lo, (size_t)m * HIDN + n, fmaxf(v[0] + b.x, 0.f), fmaxf(v[1] + b.y, 0.f),
                               fmaxf(v[2] + b.z, 0.f), fmaxf(v[3] + b.w, 0.f));
        }
    }
};
// The same layer with fp16 activations and weights in one product (no-gradient forward): `in` and `w` point at
// fp16 data of the same layouts; the outputs are the fp32 partial sums or the (hi, lo) bf16 hidden layer as above.
template <int FEAT_, int HIDN, int BM_, bool PARTIAL>
struct FcFwdF16T : FcFwdT<FEAT_, HIDN, BM_, PARTIAL> {
    static constexpr bool F16 = true;
    static constexpr int RING = 4;      // one workgroup per CU: bytes on their way hide the latency of memory
};

// categorical head: rows of the packed head matrix are the A*atoms categorical rows
// C51: atom logits fp32 [M][ZS] with bias; ZS = ZW (dense, the inference output) or the padded head width
// (the gradient step's own buffers: 16-byte stores).
template <int HIDN, int BM_>
struct HeadFwdC51 {
    static constexpr int BM = BM_, RING = 2, K = HIDN;
    static constexpr bool SHORT_K = false, WIDE = false, STORES_16BIT = false;
    static constexpr int PREFETCH_LOADS = 0;
    const __bf16 *in, *in_lo;
    int M;
    const __bf16 *w, *w_lo;
    const float *bias;   // padded head width entries (zeros past ZW)
    float *z;       // [M][ZS]
    int NHP;        // rows of the packed head matrix (multiple of 64)
    int ZW;         // A*atoms
    int ZS;         // row stride in floats: ZW, or a multiple of 64 >= ZW
    __device__ __forceinline__ const __bf16 *act() const { return in; }
    __device__ __forceinline__ const __bf16 *act_lo() const { return in_lo; }
    __device__ __forceinline__ const __bf16 *weights() const { return w; }
    __device__ __forceinline__ const __bf16 *weights_lo() const { return w_lo; }
    __device__ __forceinline__ int tiles() const { return NHP / 16; }
    __device__ __forceinline__ float4 prefetch(int, int n) const {
        return *reinterpret_cast<const float4 *>(bias + (n < NHP ? n : 0));
    }
    __device__ __forceinline__ void store(int m, int n, f32x4 v, int, float4 b) const {
        if (m >= M || n >= NHP) return;
        float *dst = z + (size_t)m * ZS + n;
        if (ZS != ZW) {                        // padded rows: every column exists
            *reinterpret_cast<float4 *>(dst) = make_float4(v[0] + b.x, v[1] + b.y, v[2] + b.z, v[3] + b.w);
        } else if ((ZW & 1) == 0) {            // dense rows of even length: n and m*ZW are even, 8-byte stores
            if (n + 1 < ZW) *reinterpret_cast<float2 *>(dst) = make_float2(v[0] + b.x, v[1] + b.y);
            if (n + 3 < ZW) *reinterpret_cast<float2 *>(dst + 2) = make_float2(v[2] + b.z, v[3] + b.w);
        } else {
            const float r[4] = {v[0] + b.x, v[1] + b.y, v[2] + b.z, v[3] + b.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < ZW) dst[e] = r[e];
        }
    }
};

// --------------------------- input gradients ------------------------------
// d(pre_fc) = (dz W_head) * [h > 0]; the contraction length is the padded head width
template <int HIDN, int BM_>
struct HeadDgrad {
    static constexpr int BM = BM_, RING = 2;
    static constexpr bool SHORT_K = true, WIDE = true;
    const __bf16 *in;    // dz [M][K]
    int M, K;
    const __bf16 *w;     // [HIDN][K]
    const __bf16 *h;
    __bf16 *out;         // [M][HIDN]
    __device__ __forceinline__ const __bf16 *act() const { return in; }
    __device__ __forceinline__ const __bf16 *weights() const { return w; }
    __device__ __forceinline__ int tiles() const { return HIDN / 16; }
    static constexpr int PREFETCH_LOADS = 2;
    struct Hidden { u32x4 w[2]; };
    __device__ __forceinline__ Hidden prefetch(int m, int n) const {
        const u32x4 *at = reinterpret_cast<const u32x4 *>(h + (size_t)(m < M ? m : 0) * HIDN + n);
        return Hidden{{at[0], at[4]}};
    }
    __device__ __forceinline__ void store(int m, int n, int half, f32x4 v, f32x4 v4, const Hidden &hidden) const {
        if (m >= M) return;
        const u32x4 hw = hidden.w[half];
        const size_t at = (size_t)m * HIDN + n;
        f32x4 a = unpack_bf16x4(u32x2{hw[0], hw[1]}), b = unpack_bf16x4(u32x2{hw[2], hw[3]});
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = a[e] > 0.f ? v[e] : 0.f;
            b[e] = b[e] > 0.f ? v4[e] : 0.f;
        }
        const u32x2 x = pack_bf16x4(a[0], a[1], a[2], a[3]), y = pack_bf16x4(b[0], b[1], b[2], b[3]);
        *reinterpret_cast<u32x4 *>(out + at) = u32x4{x[0], x[1], y[0], y[1]};
    }
};

// d(pre of the last convolution) = (d(pre_fc) W_fc) * [act > 0]      [B][FEAT], NHWC index
template <int FEAT_, int HIDN, int BM_>
struct FcDgradT {
    static constexpr int BM = BM_, RING = 2, K = HIDN, FEAT = FEAT_;
    static constexpr bool SHORT_K = false, WIDE = true;
    const __bf16 *in;         // [M][HIDN]
    int M;
    const __bf16 *w;          // [FEAT][HIDN]
    const uint8_t *maskbits;  // sign bits of the activations, bit e&7 of byte e>>3 for element e = m*FEAT + n
    __bf16 *out;
    __device__ __forceinline__ const __bf16 *act() const { return in; }
    __device__ __forceinline__ const __bf16 *weights() const { return w; }
    __device__ __forceinline__ int tiles() const { return FEAT / 16; }
    static constexpr int PREFETCH_LOADS = 1;
    // the ReLU-derivative bits of the 64 outputs (m, n / 64 * 64 ..) as one word (a wavefront's channels of a position), fetched
    // before the epilogue; FEAT is a multiple of 64, so that it holds them all or none
    __device__ __forceinline__ u32x2 prefetch(int m, int n) const {
        static_assert(FEAT % 64 == 0, "whole words");
        const size_t at = (size_t)(m < M ? m : 0) * FEAT + (n < FEAT ? n & ~63 : 0);
        return *reinterpret_cast<const u32x2 *>(maskbits + (at >> 3));
    }
    __device__ __forceinline__ void store(int m, int n, int half, f32x4 v, f32x4 v4, u32x2 bits) const {
        if (m >= M || n >= FEAT) return;
        const uint32_t mb = bits[half] >> (n & 31);
        const size_t at = (size_t)m * FEAT + n;
        const u32x2 x = pack_bf16x4(mb & 1 ? v[0] : 0.f, mb & 2 ? v[1] : 0.f, mb & 4 ? v[2] : 0.f, mb & 8 ? v[3] : 0.f);
        const u32x2 y = pack_bf16x4(mb & 16 ? v4[0] : 0.f, mb & 32 ? v4[1] : 0.f, mb & 64 ? v4[2] : 0.f, mb & 128 ? v4[3] : 0.f);
        *reinterpret_cast<u32x4 *>(out + at) = u32x4{x[0], x[1], y[0], y[1]};
    }
};

// --------------------------- weight gradients -----------------------------
// part[n][k] = sum_m dY[m][n] act(m,k); dY is a dense [M][N1] bf16 matrix.
// fc layer: its input in rows or in fragment order (LastActs)
template <int FEAT, int HIDN, int UNITS>   // UNITS: fc_wgrad_units
struct FcWgrad {
    static constexpr int BN1 = UNITS, BK2 = 64, WAVES_X = UNITS == 256 ? 1 : 2, N1 = HIDN, KP = FEAT;
    const __bf16 *in, *dy;
    int M;
    bool frag;
    // m: multiple of 32, so that both orders hold rows m .. in one piece from here on
    __device__ __forceinline__ const char *xbase(int m) const { return reinterpret_cast<const char *>(in + (size_t)m * FEAT); }
    __device__ __forceinline__ uint32_t xoff(int r, int k) const {   // k: multiple of 8
        return frag ? (uint32_t)((r >> 4) * (FEAT * 32) + (r & 15) * 16 + (k >> 5) * (FRAG_STEP * 2) + ((k & 31) >> 3) * 256)
                    : (uint32_t)(r * (FEAT * 2) + k * 2);
    }
};
// heads: N1 (padded head rows) is a run-time value
template <int HIDN>
struct HeadWgrad {
    static constexpr int BN1 = 64, BK2 = 128, WAVES_X = 4, KP = HIDN;
    const __bf16 *in, *dy;    // h [M][HIDN]
    int M, N1;
    __device__ __forceinline__ const char *xbase(int m) const { return reinterpret_cast<const char *>(in + (size_t)m * HIDN); }
    __device__ __forceinline__ uint32_t xoff(int r, int k) const { return (uint32_t)(r * (HIDN * 2) + k * 2); }
};

}  // namespace arn
