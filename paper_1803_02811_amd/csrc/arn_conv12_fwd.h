// The convolutions of the 2-convolution network in the gradient step's forward, in one kernel and in three bf16 products
// (two for conv1, whose pixel operand is exact): act1 goes to conv2 through LDS, its high part to memory for the backward
// pass.  One workgroup of eight wavefronts takes a range of samples, or -- small batches -- a band of rows of one sample's
// last feature map, recomputing the conv1 rows its windows reach into (two bands then write the same bits of act1).
//
// Both layers' weights stay in registers (64 + 64).  What bounds it at 80 samples (8.6 us): the latency of one sample's layers
// (44% of the wavefronts' cycles at a wait, LDS busy 18%, matrix cores 8%).  At 2048 samples it takes 49.6 us; the three kernels
// of this network's embedding in the 104x80 three-convolution one took 49 + 51 + 46.
#pragma once
#include "arn_infer_small.h"

namespace arn {

constexpr int C12_THREADS = 512;

struct Conv12Args {
    const uint8_t *obs;
    const __bf16 *w1, *w1_lo, *w2, *w2_lo;
    const float *b1, *b2;
    __bf16 *a1;                // act1 hi [B][P1][NC1]
    uint8_t *m1;               // sign bits of act1, mask1_bytes per sample
    __bf16 *a2, *a2_lo;        // act2 (LastActs)
    uint8_t *m2;               // sign bits of act2
    bool frag;                 // act2 in fragment order
};

template <class Geo, class P2>
__global__ __launch_bounds__(C12_THREADS) void conv12_fwd_kernel(const Conv12Args a, int B, int spw, int rows, int bands) {
    constexpr int IN_H = Geo::IN_H, IN_W = Geo::IN_W, W1 = Geo::W1, W2 = Geo::W2, OBS_BYTES = Geo::OBS_BYTES, NC1 = Geo::NC1, NC2 = Geo::NC2;
    constexpr int KS1 = KW1 / 32, KS2 = Geo::KW2 / 32, CT2 = NC2 / 16, G2 = 8 / CT2;
    constexpr int W4 = 4 * IN_W / 16;                       // 16-byte words in four rows of a channel plane
    constexpr int NL = (4 * W4 * (Geo::H1 + 1) + C12_THREADS - 1) / C12_THREADS;
    constexpr int FRAME = 2 * OBS_BYTES, IMG = P2::IMG;
    static_assert(NC1 == 16 && KS2 % 4 == 0 && layout_is_uniform<P2>() && P2::ZERO_FILL, "one channel tile in conv1, bordered image");
    static_assert(FRAME + 2 * IMG <= 160 * 1024 && FRAME % 16 == 0 && IMG % 16 == 0, "LDS budget");

    __shared__ u32x4 lds[(FRAME + 2 * IMG) / 16];
    u32x4 *const s_img = lds;                               // bf16 [4][IN_H][IN_W]
    char *const img = reinterpret_cast<char *>(lds);
    char *const a1l = img + FRAME;                          // act1 image, hi then lo

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    int s_begin, band = 0;
    if (bands > 1) band_of_block(blockIdx.x, gridDim.x, bands, s_begin, band);
    else s_begin = sample_block(blockIdx.x, gridDim.x, spw, a.frag) * spw;
    const int s_end = min(s_begin + spw, B);
    const int r2_0 = band * rows, r2_1 = min(r2_0 + rows, Geo::H2);
    const int r1_0 = max(S2 * r2_0 - Geo::PAD2, 0), r1_1 = min(S2 * (r2_1 - 1) - Geo::PAD2 + K2, Geo::H1);
    const int p1_0 = r1_0 * W1, p1_1 = r1_1 * W1, p2_0 = r2_0 * W2, p2_1 = r2_1 * W2;

    // the frame rows 4 r1_0 .. 4 (r1_1 - 1) + 7 of the four planes
    const int nw = W4 * (r1_1 - r1_0 + 1), w0 = W4 * r1_0;
    u32x4 rimg[NL];
    int word[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        int idx = tid + C12_THREADS * i;
        idx = idx < 4 * nw ? idx : 4 * nw - 1;
        const int ch = (idx >= nw) + (idx >= 2 * nw) + (idx >= 3 * nw);
        word[i] = ch * (IN_H * IN_W / 16) + w0 + idx - ch * nw;
    }
    auto gload = [&](int s) __attribute__((always_inline)) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(a.obs + (size_t)s * OBS_BYTES);
#pragma unroll
        for (int i = 0; i < NL; ++i) rimg[i] = src[word[i]];
    };
    gload(s_begin);
    bf16x8 w1h[KS1], w1l[KS1], w2h[KS2], w2l[KS2];
    const int ct = wave % CT2, t_first = wave / CT2;
    {
        const size_t r1 = frag_base(0, KW1, lane), r2 = frag_base(ct, Geo::KW2, lane);
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) {
            w1h[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(a.w1 + r1 + FRAG_STEP * ks));
            w1l[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(a.w1_lo + r1 + FRAG_STEP * ks));
        }
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) {
            w2h[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(a.w2 + r2 + FRAG_STEP * ks));
            w2l[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(a.w2_lo + r2 + FRAG_STEP * ks));
        }
    }
    const float4 bias1 = *reinterpret_cast<const float4 *>(a.b1 + 4 * lg);
    const float4 bias2 = *reinterpret_cast<const float4 *>(a.b2 + ct * 16 + 4 * lg);
    for (int i = tid; i < 2 * IMG / 16; i += C12_THREADS) lds[FRAME / 16 + i] = zero_u4();   // zero borders, written once
    bool first = true;
    for (int s = s_begin; s < s_end; ++s) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (tid + C12_THREADS * i < 4 * nw) {
                s_img[2 * word[i]] = u8x8_to_bf16x8(rimg[i].x, rimg[i].y);
                s_img[2 * word[i] + 1] = u8x8_to_bf16x8(rimg[i].z, rimg[i].w);
            }
        }
        if (first) wait_global_loads();      // the weights, once: not to be waited for behind the next frame's loads
        first = false;
        __syncthreads();                     // frame staged; every conv2 read of the act1 image done
        if (s + 1 < s_end) gload(s + 1);

        // ---- conv1: frame image -> act1 image and memory ----
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
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) {
                const bf16x8 b = as_bf16x8(u32x4{f[2 * ks].x, f[2 * ks].y, f[2 * ks + 1].x, f[2 * ks + 1].y});
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1l[ks], b, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1h[ks], b, acc, 0, 0, 0);
            }
            constexpr float sc = 1.0f / 255.0f;
            const float r0 = fmaxf(acc[0] * sc + bias1.x, 0.f), r1 = fmaxf(acc[1] * sc + bias1.y, 0.f);
            const float r2 = fmaxf(acc[2] * sc + bias1.z, 0.f), r3 = fmaxf(acc[3] * sc + bias1.w, 0.f);
            const bf16x4 h = {(__bf16)r0, (__bf16)r1, (__bf16)r2, (__bf16)r3};
            const u32x2 hi = __builtin_bit_cast(u32x2, h);
            const u32x2 lo = pack_bf16x4(r0 - (float)h[0], r1 - (float)h[1], r2 - (float)h[2], r3 - (float)h[3]);
            const uint32_t bits = sign_bits16(r0, r1, r2, r3, lg);     // all lanes take part
            if (valid) {
                char *dst = a1l + P2::dst_off(pos) + 8 * lg;
                *reinterpret_cast<u32x2 *>(dst) = hi;
                *reinterpret_cast<u32x2 *>(dst + IMG) = lo;
                *reinterpret_cast<u32x2 *>(a.a1 + ((size_t)s * Geo::P1 + pos) * NC1 + 4 * lg) = hi;
                if (lg == 0) *reinterpret_cast<uint16_t *>(a.m1 + (size_t)s * mask1_bytes(Geo::P1, NC1) + pos * 2) = (uint16_t)bits;
            }
        }
        __syncthreads();                     // act1 complete; every read of the frame image done

        // ---- conv2: act1 image -> memory ----
#pragma unroll 1
        for (int t = t_first; p2_0 + t * 16 < p2_1; t += G2) {
            int pos = p2_0 + t * 16 + li;
            const bool valid = pos < p2_1;
            pos = valid ? pos : p2_1 - 1;
            const char *src = a1l + P2::base_off(pos) + P2::lane_off(lg);
            bf16x8 fh[KS2], fl[KS2];
#pragma unroll
            for (int ks = 0; ks < KS2; ++ks) {
                fh[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(src + P2::step_off(ks)));
                fl[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(src + IMG + P2::step_off(ks)));
            }
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS2; ++ks) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2l[ks], fh[ks], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2h[ks], fl[ks], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2h[ks], fh[ks], acc, 0, 0, 0);
            }
            const float r0 = fmaxf(acc[0] + bias2.x, 0.f), r1 = fmaxf(acc[1] + bias2.y, 0.f);
            const float r2 = fmaxf(acc[2] + bias2.z, 0.f), r3 = fmaxf(acc[3] + bias2.w, 0.f);
            const uint32_t bits = sign_bits16(r0, r1, r2, r3, lg);
            if (valid) {
                const int n = ct * 16 + 4 * lg;
                store_bf16x4_split(a.a2, a.a2_lo, LastActs<NC2, Geo::P2>::at(a.frag, s, pos, n), r0, r1, r2, r3, std::true_type());
                if (lg == 0) *reinterpret_cast<uint16_t *>(a.m2 + (((size_t)s * Geo::P2 + pos) * NC2 + ct * 16) / 8) = (uint16_t)bits;
            }
        }
    }
}

}  // namespace arn
