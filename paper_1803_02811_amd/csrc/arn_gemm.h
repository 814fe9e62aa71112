// MFMA building blocks for gfx950: two workgroup-level contraction kernels that
// the dense layers (fc, categorical head) are instances of.
//
//   gemm_nt_body : out[m][n] = sum_k act(m,k) * W[n][k]
//       forward layers and input gradients; W is packed in fragment order.
//   gemm_tn_body : out[n][k] = sum_m dY[m][n] * act(m,k)
//       weight gradients: the contraction runs over the batch/position index,
//       which is the slow index of both operands in memory, so fragments are
//       taken from LDS with the transposing read ds_read_b64_tr_b16.
//
// MFMA operand layouts (checked on hardware):
//   16x16x32  A (16 x 32): lane l holds row l%16, k = 8*(l/16) .. +7;  B (32 x 16): lane l holds col l%16, same k;
//             D (16 x 16): lane l holds col l%16, rows 4*(l/16) + r, r = 0..3
//   32x32x16  A (32 x 16): lane l holds row l%32, k = 8*(l/32) .. +7;  B (16 x 32): lane l holds col l%32, same k;
//             D (32 x 32): lane l holds col l%32, rows 8*(r/4) + 4*(l/32) + r%4, r = 0..15
// The weights (or dY) go in as A and the activations as B, so a lane ends up
// with 4 consecutive channels of one position: one 8-byte NHWC store.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace arn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
// 16- and 8-byte register/LDS words as native vectors (plain loads and stores, kept in registers)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

__device__ __forceinline__ u32x2 pack_bf16x4(float a, float b, float c, float d) {
    bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    return __builtin_bit_cast(u32x2, v);
}

// v -> (hi, lo) with hi = bf16(v), lo = bf16(v - hi)
template <bool ALWAYS_LO = false>
__device__ __forceinline__ void store_bf16x4_split(__bf16 *hi, __bf16 *lo, size_t at, float a, float b, float c,
                                                   float d, std::integral_constant<bool, ALWAYS_LO> = {}) {
    const bf16x4 h = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    *reinterpret_cast<u32x2 *>(hi + at) = __builtin_bit_cast(u32x2, h);
    if (ALWAYS_LO || lo) {
        const bf16x4 l = {(__bf16)(a - (float)h[0]), (__bf16)(b - (float)h[1]), (__bf16)(c - (float)h[2]),
                          (__bf16)(d - (float)h[3])};
        *reinterpret_cast<u32x2 *>(lo + at) = __builtin_bit_cast(u32x2, l);
    }
}

// ReLU sign bits of a 16x16 MFMA tile: lane (li = l%16, lg = l/16) holds channels 4*lg..4*lg+3
// of position li; the four lanes of a position combine their nibbles into one 16-bit word
// (bit c = value of channel c > 0), valid in every participating lane.
__device__ __forceinline__ uint32_t sign_bits16(float a, float b, float c, float d, int lg) {
    uint32_t t = ((a > 0.f ? 1u : 0u) | (b > 0.f ? 2u : 0u) | (c > 0.f ? 4u : 0u) | (d > 0.f ? 8u : 0u)) << (4 * lg);
    // v_permlane16_swap / v_permlane32_swap (VALU, no LDS traffic): with both operands equal, the two
    // results are the lane's own value and that of the lane 16 (32) away (checked on hardware)
    const auto a16 = __builtin_amdgcn_permlane16_swap(t, t, false, false);
    t = a16[0] | a16[1];
    const auto a32 = __builtin_amdgcn_permlane32_swap(t, t, false, false);
    return a32[0] | a32[1];
}

// relu(v) as the bf16 pair (hi, lo), four channels
__device__ __forceinline__ void relu_split(f32x4 v, u32x2 &hi, u32x2 &lo) {
    const float r0 = fmaxf(v[0], 0.f), r1 = fmaxf(v[1], 0.f), r2 = fmaxf(v[2], 0.f), r3 = fmaxf(v[3], 0.f);
    hi = pack_bf16x4(r0, r1, r2, r3);
    lo = pack_bf16x4(r0 - __uint_as_float(hi.x << 16), r1 - __uint_as_float(hi.x & 0xffff0000u), r2 - __uint_as_float(hi.y << 16),
                     r3 - __uint_as_float(hi.y & 0xffff0000u));
}
// which of eight bf16 are positive, bit i for value i
__device__ __forceinline__ uint32_t positive_bits(u32x4 v) {
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    uint32_t z = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const s16x2 w = __builtin_bit_cast(s16x2, (uint32_t)v[i]), zero = {0, 0}, one = {1, 1};
        z |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_elementwise_max(w, zero), one)) << (2 * i);
    }
    return (z | z >> 15) & 0xff;     // even values' bits in the lower half, odd ones' in the upper
}
// The value, as the compiler sees it a new one each time: what is computed from it is computed where it is used, not kept in
// registers across a loop.
__device__ __forceinline__ int recomputed(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ f32x4 unpack_bf16x4(u32x2 u) {
    bf16x4 v = __builtin_bit_cast(bf16x4, u);
    f32x4 r = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
    return r;
}

// eight uint8 (two little-endian words) -> eight bf16, exact
__device__ __forceinline__ u32x4 u8x8_to_bf16x8(uint32_t lo, uint32_t hi) {
    auto two = [](uint32_t b0, uint32_t b1) -> uint32_t {
        return (__float_as_uint((float)b0) >> 16) | (__float_as_uint((float)b1) & 0xffff0000u);
    };
    u32x4 r;
    r.x = two(lo & 0xff, (lo >> 8) & 0xff);
    r.y = two((lo >> 16) & 0xff, lo >> 24);
    r.z = two(hi & 0xff, (hi >> 8) & 0xff);
    r.w = two((hi >> 16) & 0xff, hi >> 24);
    return r;
}

// Weights that a wavefront keeps in registers as MFMA A-operand fragments (16 rows x 32 k) are packed in fragment
// order: the eight values of lane l for (16-row tile t, k-step ks) of a [rows][K] matrix are the 16 contiguous
// bytes at element ((t * K/32 + ks) * 64 + l) * 8.  A wavefront's load of one fragment is then one contiguous
// kilobyte; read from the row-major matrix it was sixteen 64-byte pieces a row apart, and a workgroup's
// 300 KB of such loads took 8 us before the first MFMA (measured).  frag_base + FRAG_STEP * ks addresses it.
constexpr int FRAG_STEP = 512;
__device__ __forceinline__ size_t frag_base(int tile, int K, int lane) { return (size_t)tile * K * 16 + (size_t)lane * 8; }
// the same index for the packing side: element (row, k) of the [rows][K] matrix
__host__ __device__ constexpr long frag_index(long row, long k, long K) {
    return ((row >> 4) * (K >> 5) + (k >> 5)) * 512 + ((((k & 31) >> 3) << 4) + (row & 15)) * 8 + (k & 7);
}

// Workgroups go to the eight XCDs round robin.  This renumbers blocks 0 .. n-1 so that an XCD gets runs of `run` (a power of
// two) consecutive ones: data that neighbouring blocks write side by side in a cache line then meets in one L2.
__device__ __forceinline__ int xcd_runs(int b, int n, int run) {
    int base = 0;
    for (; run > 1; run >>= 1) {
        const int chunk = 8 * run, full = (n - base) / chunk * chunk;
        if (b - base < full) {
            const int r = (b - base) % chunk;
            return b - r + (r & 7) * run + (r >> 3);
        }
        base += full;
    }
    return b;
}
// sample range of `spw` samples that workgroup b of n works on: with the activations in fragment order the 16-byte words of
// eight consecutive samples share a cache line (256 samples, a workgroup each: 10.2 -> 9.4 us for the three convolutions)
__device__ __forceinline__ int sample_block(int b, int n, int spw, bool frag) {
    return frag ? xcd_runs(b, n, spw == 1 ? 8 : spw == 2 ? 4 : 1) : b;
}

// Addresses (in elements) of the last convolution's activations [sample][position][NC channels], the fc layer's input:
// rows, or -- for the batches that fc_small_kernel serves -- fragment order over (sample, position * NC + channel).
template <int NC, int P>
struct LastActs {
    static_assert(NC % 32 == 0, "whole k-steps per position");
    template <bool FRAG>
    static __device__ __forceinline__ size_t at(int s, int pos, int n) {   // n: multiple of 4
        if constexpr (FRAG)
            return (size_t)(s >> 4) * (NC * P * 16) + (s & 15) * 8 + (size_t)(pos * (NC * 16) + (n >> 5) * FRAG_STEP + ((n & 31) >> 3) * 128 + (n & 7));
        else
            return ((size_t)s * P + pos) * NC + n;
    }
    static __device__ __forceinline__ size_t at(bool frag, int s, int pos, int n) { return frag ? at<true>(s, pos, n) : at<false>(s, pos, n); }
};

__device__ __forceinline__ u32x4 zero_u4() { return u32x4{0u, 0u, 0u, 0u}; }

// Waits until every global load of this wavefront has returned (s_waitcnt vmcnt(0), other counters unchanged).
// Kernels that keep weights in registers call it once after loading them: otherwise the compiler places the
// wait for those loads at their first use inside the sample loop, where it cannot tell them from the prefetch
// of the next sample issued just before -- and every iteration would wait for its own prefetch.
__device__ __forceinline__ void wait_global_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Copies 16 bytes per lane from base + voff (base wavefront-uniform) to LDS byte offset lds_off + 16 * lane (lds_off
// wavefront-uniform), without passing through registers.  It counts as a vector memory operation (wait_global_loads, vmcnt);
// the compiler does not know of it, so the caller waits before the data is read and before the kernel ends.
// m0 holds the LDS offset and is lost: a value the compiler has put there is set again before its next use.  (The warning is
// that the compiler does not save a reserved register around the statement, which nothing here asks of it.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy_to_lds(const void *base, uint32_t voff, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_off), "v"(voff), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ uint32_t lds_offset(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
// waits until at most N vector memory operations of this wavefront are outstanding
template <int N>
__device__ __forceinline__ void wait_vmem() {
    static_assert(N >= 0 && N < 64, "six-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// ---------------------------------------------------------------------------
// out[m][n] = sum_k act(m,k) W[n][k]
//
// Problem P supplies
//   BM               positions per workgroup tile: 32, 64 or 128 (128 channels)
//   RING             pairs of 32-wide stages in LDS: 2 or 4
//   SHORT_K          whether a contraction range may be shorter than RING pairs
//   K                contraction length, multiple of 64 (static or a data member)
//   M                rows of act (rows past the end are read from the last one and dropped by store)
//   act(), act_lo()  act, row-major 16-bit values [M][K]
//   weights(), weights_lo()   W in fragment order (frag_index)
//   tiles()          16-row tiles of W (even); tiles past the end are read from the last one and dropped by store
//   WIDE             whether store takes eight channels instead of four
//   prefetch(m, n)                   what the epilogue of an output reads (bias, sign of an activation), loaded before the
//                                    k loop: a load in the epilogue would be waited for once per output
//   store(m, n, v, z, prefetched)    epilogue for channels n..n+3 of position m
//   STORES_16BIT                     not WIDE: whether that writes 16-bit values or fp32, which decides the order of the stores
//   prefetch(m, n)                   WIDE: the same for channels n..n+7 and n+32..n+39, what a lane has of a position
//   PREFETCH_LOADS                   WIDE: vector memory loads that prefetch() compiles to.  Never more than there are: the waits
//                                    for the last copies leave that many operations outstanding, so one too many and fragments
//                                    are read before they have arrived.  Checked to be the fewest that its result can take
//   store(m, n, half, v, v4, prefetched)   WIDE: for channels n..n+7, the prefetched first (half 0) or second eight
// Grid: x = position tiles, y = channel tiles, z = range of the contraction (problems with a member ksplit).
//
// SPLIT = true is the three-product bf16 scheme of the gradient step's forward: each operand is a pair (hi, lo) of bf16 with
// hi + lo carrying ~16 mantissa bits, and the product is accumulated as lo_w*hi_a + hi_w*lo_a + hi*hi in fp32.
//
// Four wavefronts, each 64 channels x BM/2 positions.  A stage is 32 of the contraction.  Operands are copied from memory
// straight to LDS (no registers, no conversion, no write instructions), up to 2 * RING stages ahead of their use, and a
// wavefront's fragments of stage s+1 are read from LDS between its MFMAs on stage s.  The order of the words in LDS makes
// the fragment reads conflict-free under the bank rule of arn_resident_conv.h; the copies apply it to their source address.
//
// What bounds it: with three products the matrix cores come nearest (busy 60% of a launch's cycles at 8192 samples, 48% at
// 2048; LDS 20 and 16%; the chip's power limit sets the clock, 1.7 - 1.9 GHz here, which is also why the MFMAs are 16x16x32:
// 32x32x16 ran the same loop in fewer cycles at a lower clock, 58 against 55 us); with one product nothing is near its rate
// (matrix cores 38%, LDS 19% at 8192 samples) and wavefronts wait, for the copies at the start of a range and at every
// stage's barrier (35% of their cycles at a wait).  Measured before (operands through registers, one stage ahead) and after, us:
// fc forward of 8192 samples, three products 87 -> 65; of 2048 samples 26.7 -> 22.6; one product, 8192 samples 41 -> 35;
// categorical head of 8192 samples and 960 rows 35 -> 32, its input gradient 19.4 -> 15.5.
// ---------------------------------------------------------------------------
// Problems with a data member `ksplit` cut the contraction into that many
// ranges, one per blockIdx.z; their store() receives z and writes a
// partial sum that a later kernel adds up in z order.
template <class P, class = void>
struct HasKSplit {
    static constexpr bool value = false;
};
template <class P>
struct HasKSplit<P, decltype((void)P::ksplit)> {
    static constexpr bool value = true;
};
// Problems with a static member F16 = true hold fp16 operands (same 16-byte fragments, the fp16 MFMA): the single
// product of the forward passes that carry no gradient.
template <class P, class = void>
struct IsF16 {
    static constexpr bool value = false;
};
template <class P>
struct IsF16<P, decltype((void)P::F16)> {
    static constexpr bool value = P::F16;
};
template <bool F16>
__device__ __forceinline__ f32x4 mfma_16x16x32(u32x4 a, u32x4 b, f32x4 c) {
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}
constexpr int NT_THREADS = 256, NT_BN = 128;
template <int N>
using Count = std::integral_constant<int, N>;
// LDS bytes of gemm_nt_body<P, SPLIT>
template <class P, bool SPLIT = false>
constexpr int gemm_nt_lds_bytes() { return P::RING * 2 * (P::BM + NT_BN) * 64 * (SPLIT ? 2 : 1); }

// The work of workgroup (bx, by, bz) of a grid of gx x gy x gz workgroups, in the caller's LDS buffer.
template <class P, bool SPLIT = false>
__device__ __forceinline__ void gemm_nt_body(u32x4 *lds, const P &p, int bx, int by, int bz, int gx, int gy, int gz) {
    constexpr int BM = P::BM, PARTS = SPLIT ? 2 : 1, RING = P::RING;
    constexpr int MB = BM / 32;                                  // position tiles of 16 per wavefront; four channel tiles
    constexpr int GA = BM / 32;                                  // 8-row groups of act a wavefront copies per pair of stages and part
    static_assert(BM == 32 || BM == 64 || BM == 128, "tile shape");
    static_assert(RING == 2 || RING == 4, "slots");
    int st_begin = 0, st_end = p.K / 32;
    if constexpr (HasKSplit<P>::value) {
        // Split-k launches: workgroups go to the eight XCDs round robin in linear order (x fastest), and each XCD has
        // an L2 of its own.  With the plain mapping an XCD sees every k range of its position tiles and all of W;
        // remapped, an XCD works on one k range (or a few) of a band of position tiles, so what its L2 fetches from
        // memory is halved (measured: 77.2 -> 38.6 MB per launch of the fc layer at 2048 samples).  Only for grids that
        // split evenly; otherwise the plain mapping.
        const bool pow2 = (gz & (gz - 1)) == 0;
        if (pow2 && gz >= 8) {
            const int L = bx + gx * (by + gy * bz), c = L & 7, zpc = gz >> 3;
            int r = L >> 3;
            bz = c * zpc + r % zpc;
            r /= zpc;
            bx = r % gx;
            by = r / gx;
        } else if (pow2 && gz > 1 && gx % (8 / gz) == 0) {
            const int L = bx + gx * (by + gy * bz), c = L & 7, g = 8 / gz, xs = gx / g, r = L >> 3;
            bz = c / g;
            bx = (c % g) * xs + r % xs;
            by = r / xs;
        }
        const int pairs = st_end / 2;                            // an even number of stages each, at least two
        st_begin = bz * pairs / p.ksplit * 2;
        st_end = (bz + 1) * pairs / p.ksplit * 2;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int wn = wave & 1, wm = wave >> 1;
    const int m0 = bx * BM, n0 = by * NT_BN, z = bz;
    const int NS = st_end - st_begin;

    // Sources of this wavefront's copies: GA groups of 8 rows x 64 k of act, two 16-row x 32-k tiles of W.  An activation
    // group is copied for two stages at once (whole 128-byte lines): word c of row r is stored at c ^ ((r >> 1) & 7).
    uint32_t a_off[GA], a_dst[GA];
#pragma unroll
    for (int i = 0; i < GA; ++i) {
        const int g = wave * GA + i, row = g * 8 + (lane >> 3);
        a_off[i] = (uint32_t)(min(row, p.M - 1 - m0) * p.K * 2 + ((lane & 7) ^ ((row >> 1) & 7)) * 16);
        a_dst[i] = g * 1024;
    }
    // W: a wavefront copies the two tiles of a group of 32 channels.  WIDE problems give row i of tile t of the group channel
    // 8 * (i / 4) + 4 * t + i % 4, so that a lane's two quads are eight consecutive channels: one 16-byte store of bf16.
    const int w_tile = min(n0 / 16 + wave * 2, p.tiles() - 2);
    uint32_t w_off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int ch = P::WIDE ? 8 * (li >> 2) + 4 * i + (li & 3) : 16 * i + li;
        w_off[i] = (uint32_t)((ch >> 4) * (p.K / 32) * (FRAG_STEP * 2) + lg * 256 + (ch & 15) * 16);
    }
    const char *a_src[PARTS], *w_src[PARTS];
    a_src[0] = reinterpret_cast<const char *>(p.act()) + (size_t)m0 * p.K * 2 + (size_t)st_begin * 64;
    if constexpr (SPLIT) a_src[1] = reinterpret_cast<const char *>(p.act_lo()) + (size_t)m0 * p.K * 2 + (size_t)st_begin * 64;
    const size_t w_at0 = ((size_t)w_tile * (p.K / 32) + st_begin) * (FRAG_STEP * 2);
    w_src[0] = reinterpret_cast<const char *>(p.weights()) + w_at0;
    if constexpr (SPLIT) w_src[1] = reinterpret_cast<const char *>(p.weights_lo()) + w_at0;
    const uint32_t lds0 = lds_offset(lds);
    constexpr int A_PAIR = BM * 128, W_STAGE = NT_BN * 64, W_BASE = RING * PARTS * A_PAIR;   // LDS: RING pairs of act, then of W
    constexpr int A_COPIES = GA * PARTS, W_COPIES = 2 * PARTS, PAIR_COPIES = A_COPIES + 2 * W_COPIES;
    auto copy_a = [&](int s, int c) __attribute__((always_inline)) {                         // stages s and s+1, s even
        const int part = c / GA, i = c % GA;
        copy_to_lds(a_src[part] + (size_t)s * 64, a_off[i], lds0 + ((s >> 1) & (RING - 1)) * (PARTS * A_PAIR) + part * A_PAIR + a_dst[i]);
    };
    auto copy_w = [&](int s, int c) __attribute__((always_inline)) {
        const int part = c >> 1, i = c & 1;
        copy_to_lds(w_src[part] + (size_t)s * (FRAG_STEP * 2), w_off[i],
                    lds0 + W_BASE + ((s & (2 * RING - 1)) * PARTS + part) * W_STAGE + (wave * 2 + i) * 1024);
    };

    // the lane's outputs: QUADS quads (1, or 2 neighbouring ones) at channel n_of(a) of position m_of(b)
    constexpr int QUADS = P::WIDE ? 2 : 1;
    const auto m_of = [&](int b) { return m0 + (wm * MB + b) * 16 + li; };
    const auto n_of = [&](int a) { return n0 + (wn * 4 + a) * 16 + 4 * QUADS * lg; };
    decltype(p.prefetch(0, 0)) pre[P::WIDE ? 1 : 4][MB];
    auto prefetch_all = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < (P::WIDE ? 1 : 4); ++a)
#pragma unroll
            for (int b = 0; b < MB; ++b) pre[a][b] = p.prefetch(m_of(b), n_of(a));
    };
    // What WIDE problems read per position comes from memory, not from the L2, and loads return in order: ahead of the first
    // copies it would hold up the first stage.  It is asked for when the last copies have been.  (fc input gradient alone, with one
    // word instead of eight single bytes per lane: 16.0 -> 14.7 us at 2048 samples, 49.9 -> 46.0 at 8192.  Tiles below 128 positions and the
    // eight stages of the 2-convolution network: ahead of the first copies, right behind them or here, whole steps are within 0.4%, but
    // right behind them costs 104x80 0.7 to 1% at 200 and 255 samples.)
    constexpr int LATE = MB * P::PREFETCH_LOADS;
    static_assert(!P::WIDE || P::PREFETCH_LOADS == (sizeof(pre[0][0]) + 15) / 16, "what a load brings at most: 16 bytes");
    if constexpr (!P::WIDE) prefetch_all();
#pragma unroll
    for (int s = 0; s < 2 * RING; s += 2)
        if (s < NS) {
#pragma unroll
            for (int c = 0; c < W_COPIES; ++c) copy_w(s, c);
#pragma unroll
            for (int c = 0; c < A_COPIES; ++c) copy_a(s, c);
#pragma unroll
            for (int c = 0; c < W_COPIES; ++c) copy_w(s + 1, c);
        }

    f32x4 acc[4][MB];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // fragments of a stage in the order they are read: per part, MB of act and four of W
    constexpr int READS = (MB + 4) * PARTS, MFMAS = 4 * MB * (SPLIT ? 3 : 1);
    struct Frags { u32x4 f[READS]; };
    const int row = wm * (MB * 16) + li, w_at = wn * 4096 + lane * 16;
    const int a_at = row * 128 + ((lg ^ ((row >> 1) & 7)) * 16);     // of the even stage; the odd one's words are 4 further: ^ 64
    auto read_one = [&](int s, int r, Frags &f) __attribute__((always_inline)) {
        const int part = r / (MB + 4), e = r % (MB + 4);
        const char *at = reinterpret_cast<const char *>(lds);
        if (e < MB) at += ((s >> 1) & (RING - 1)) * (PARTS * A_PAIR) + part * A_PAIR + (a_at ^ ((s & 1) * 64)) + e * 2048;
        else at += W_BASE + ((s & (2 * RING - 1)) * PARTS + part) * W_STAGE + w_at + (e - MB) * 1024;
        f.f[r] = *reinterpret_cast<const u32x4 *>(at);
    };
    auto multiply_one = [&](int q, const Frags &f) __attribute__((always_inline)) {      // no MFMA waits for the previous one
        const int t = SPLIT ? q / (4 * MB) : 2, a = q % (4 * MB) / MB, b = q % MB;
        acc[a][b] = mfma_16x16x32<IsF16<P>::value>(f.f[(t == 0 ? (PARTS - 1) * (MB + 4) : 0) + MB + a],
                                                   f.f[(t == 1 ? (PARTS - 1) * (MB + 4) : 0) + b], acc[a][b]);
    };
    // Stage s, whose fragments are in `cur`: wait until at most AHEAD copies are outstanding, so that stage s+1 has
    // arrived; then its fragments are read between the MFMAs of s.  In the steady state every stage also issues the copies
    // that take its slot (everyone has read it by then): W of stage s + 2*RING, and after odd stages the pair of act.
    auto stage = [&](auto ahead, auto w_copies, auto a_copies, int s, const Frags &cur, Frags &next) __attribute__((always_inline)) {
        constexpr int WC = decltype(w_copies)::value, COPIES = WC + decltype(a_copies)::value;
        wait_vmem<decltype(ahead)::value>();
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        int q = 0, c = 0;
#pragma unroll
        for (int r = 0; r < READS; ++r) {
            read_one(s + 1, r, next);
            for (; c < (r + 1) * COPIES / READS; ++c) {
                if (c < COPIES - WC) copy_a(s + 2 * RING - 1, c);
                else copy_w(s + 2 * RING, c - (COPIES - WC));
            }
            for (; q < (r + 1) * MFMAS / READS; ++q) multiply_one(q, cur);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // 16-bit outputs: a position's channels one after the other, a cache line holds the 64 of a wavefront; the fc layer's hidden units
    // of 8192 samples, channel group by channel group, cost 1.4 us a launch (65.4 / 64.0, one
    // product 35.0 / 33.6) and 31 MB of writes instead of 16; the categorical step of 8192 samples took 1052.5 us, now 1046.9.
    // fp32 rows: channel group by channel group; in the order of 16-bit outputs the fc layer's partials of 512 samples of 104x80 took
    // 8.6 instead of 8.2 us (one product), the head kernel that reads them 9.3 instead of 9.1, and the A2C gradient at 2048 samples of
    // 84x84 241.5 instead of 239.5.
    auto store_all = [&]() __attribute__((always_inline)) {
        if constexpr (P::WIDE) {
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int a = 0; a < 4; a += 2) p.store(m_of(b), n_of(a), a / 2, acc[a][b], acc[a + 1][b], pre[0][b]);
        } else if constexpr (P::STORES_16BIT) {
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) p.store(m_of(b), n_of(a), acc[a][b], z, pre[a][b]);
        } else {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < MB; ++b) p.store(m_of(b), n_of(a), acc[a][b], z, pre[a][b]);
        }
    };
    Frags fa, fb;
    if constexpr (P::SHORT_K) {
        if (NS < 2 * RING) {                                     // fewer stages than slots: everything is in LDS at once
            if constexpr (P::WIDE) prefetch_all();
            wait_vmem<0>();
            __syncthreads();
            for (int s = 0; s < NS; ++s) {
#pragma unroll
                for (int r = 0; r < READS; ++r) read_one(s, r, fa);
#pragma unroll
                for (int q = 0; q < MFMAS; ++q) multiply_one(q, fa);
            }
            store_all();
            return;
        }
    }
    wait_vmem<(RING - 1) * PAIR_COPIES + W_COPIES>();
    __syncthreads();
#pragma unroll
    for (int r = 0; r < READS; ++r) read_one(0, r, fa);
    int s = 0;
    for (; s + 2 * RING < NS; s += 2) {
        stage(Count<(RING - 1) * PAIR_COPIES>(), Count<W_COPIES>(), Count<0>(), s, fa, fb);
        stage(Count<(RING - 2) * PAIR_COPIES + 2 * W_COPIES>(), Count<W_COPIES>(), Count<A_COPIES>(), s + 1, fb, fa);
    }
    if constexpr (P::WIDE) prefetch_all();
    auto last_pair = [&](auto left) __attribute__((always_inline)) {    // `left` pairs follow this one
        constexpr int N = decltype(left)::value;
        stage(Count<N * PAIR_COPIES + LATE>(), Count<0>(), Count<0>(), s, fa, fb);
        stage(Count<(N - 1) * PAIR_COPIES + W_COPIES + LATE>(), Count<0>(), Count<0>(), s + 1, fb, fa);
        s += 2;
    };
    if constexpr (RING > 2) {
        last_pair(Count<3>());
        last_pair(Count<2>());
    }
    last_pair(Count<1>());
    stage(Count<LATE>(), Count<0>(), Count<0>(), s, fa, fb);
#pragma unroll
    for (int q = 0; q < MFMAS; ++q) multiply_one(q, fb);
    store_all();
}

template <class P, bool SPLIT = false>
constexpr int gemm_nt_wgs() { return 160 * 1024 / gemm_nt_lds_bytes<P, SPLIT>(); }
// The number of workgroups per CU is stated to the compiler, so that it does not save registers it has.
template <class P, bool SPLIT = false>
__global__ __launch_bounds__(NT_THREADS) __attribute__((amdgpu_waves_per_eu(gemm_nt_wgs<P, SPLIT>(), gemm_nt_wgs<P, SPLIT>())))
void gemm_nt_kernel(const P p) {
    __shared__ u32x4 lds[gemm_nt_lds_bytes<P, SPLIT>() / 16];
    gemm_nt_body<P, SPLIT>(lds, p, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x, gridDim.y, gridDim.z);
}

// ---------------------------------------------------------------------------
// part[split][n][k] = sum_{m in split} dY[m][n] * act(m,k)       (fp32)
// part[split][N1*KP + n] = sum_{m in split} dY[m][n]             (bias gradient)
//
// Problem P supplies
//   BN1, BK2         output tile (dY channels x act columns), multiples of 64
//   WAVES_X          wavefronts along act columns (1, 2 or 4)
//   N1, KP           full output shape (rows, columns; static or data members)
//   dy               dY, row-major bf16 [M][N1]
//   xbase(m), xoff(r, k)    address of act row m (a multiple of 32), byte offset of act(m + r, k .. k+7) from it, r < 32
//   int M            number of contraction rows
// Each split covers `rows_per_split` (a multiple of 64) consecutive m; partials are summed by reduce_all_kernel in split
// order, which fixes the rounding order.
//
// A stage is 32 rows.  Both operands are copied from memory straight to LDS, RING - 1 stages ahead of their use, and read
// back as fragments by transposing reads; one barrier per stage.  A transposing read takes 64 contiguous bytes of each of
// four consecutive rows, which is conflict-free when the four are 64 bytes apart modulo 256: rows are not padded (a copy
// fills 1 KB), so row r's 64-byte blocks are stored permuted, and the copies apply that to their source address.
//
// What bounds it: latency.  At 8192 samples its MFMAs would take 11 us at 2.4 GHz, and so would its LDS reads at 128 bytes per clock of a
// CU (two 8-byte reads of a wavefront per 32x32x16 MFMA with 64 x 64 outputs per wavefront, FcWgrad of large batches; three with 64 x 32);
// alone the range takes 49 (64 x 32: 64; at 2048 samples 18.3 and 20.8).  In the launch it is a part of
// (dense_backward_kernel, 2048 samples with 64 x 32 and 8192 with 64 x 64) the matrix cores are busy 22 and 28% of the cycles, LDS 14 and
// 15%, a hundredth of that bank conflicts; wavefronts spend 38 and 34% at a wait, 32 and 37% waiting to issue.  With operands through
// registers, one 64-row tile ahead, the staging writes came on top and every tile had two barriers.  Steps before / after, us: ppo of 4096
// samples 440 / 431, c51 of 8192 samples 1128 / 1111, a2c of 2048 samples 247 / 244.
// ---------------------------------------------------------------------------
constexpr int TN_ROWS = 32;
template <class P>
constexpr int gemm_tn_stage_bytes() { return TN_ROWS * (P::BN1 + P::BK2) * 2; }
// position of the 16-byte words of row r (of ROWB bytes): word c is stored at c ^ tn_swizzle(r).  Unchanged by r + 4.
template <int ROWB>
__device__ __forceinline__ int tn_swizzle(int r) { return ROWB == 128 ? (r & 2) << 1 : (r & 3) << 2; }

// Transposing LDS fragment read.
//
// `tile` holds rows (contraction index m) of ROWB bytes, their words permuted by tn_swizzle.  Returns, for MFMA lane l, the
// eight values
//   tile[mbase + 8*(l/32) + e][col0 + l%32],  e = 0..7
// i.e. an A- or B-operand fragment whose k index is the tile's row index.
// ds_read_b64_tr_b16 works on groups of 16 lanes: lane 4q+e of a group receives
// element e of the four 8-byte rows addressed by lanes q, q+4, q+8, q+12.
template <int ROWB>
__device__ __forceinline__ bf16x8 tr_fragment(const char *tile, int mbase, int col0, int lane) {
    const int o = lane & 15, G = lane >> 4;
    const int row = 8 * (G >> 1) + (o >> 2);
    const int col = col0 + 16 * (G & 1) + 4 * (o & 3);
    const char *addr = tile + mbase * ROWB + row * ROWB + ((col * 2) ^ (tn_swizzle<ROWB>(row) * 16));
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(addr));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(addr + 4 * ROWB));
    s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// The work of workgroup (bx, by, split) of 256 threads, in the caller's LDS buffer of RING * gemm_tn_stage_bytes<P>().
template <class P, int RING>
__device__ __forceinline__ void gemm_tn_body(u32x4 *lds, const P &p, float *__restrict__ part, int rows_per_split, int bx, int by,
                                             int split) {
    constexpr int BN1 = P::BN1, BK2 = P::BK2, WX = P::WAVES_X, WY = 4 / WX;
    constexpr int TY = BN1 / (32 * WY), TX = BK2 / (32 * WX);
    constexpr int YB = BN1 * 2, XB = BK2 * 2, Y_BYTES = TN_ROWS * YB, STAGE = gemm_tn_stage_bytes<P>();
    constexpr int YC = YB / 16, XC = XB / 16;                    // 16-byte words per row
    constexpr int Y_COPIES = Y_BYTES / 4096, X_COPIES = TN_ROWS * XB / 4096, COPIES = Y_COPIES + X_COPIES;   // per wavefront
    static_assert(RING >= 3 && RING <= 5 && YB % 128 == 0 && XB % 128 == 0, "slots; rows of whole 128 bytes");
    static_assert(TY >= 1 && TX >= 1 && Y_COPIES >= 1 && X_COPIES >= 1, "tile shape");
    static_assert(256 % YC == 0 && (256 / YC) * BN1 * 4 <= RING * STAGE, "bias-gradient scratch");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wx = wave % WX, wy = wave / WX;
    const int x0 = bx * BK2, y0 = by * BN1;
    const int m_begin = split * rows_per_split, m_end = min(m_begin + rows_per_split, p.M);
    const int stages = m_begin < m_end ? (m_end - m_begin + TN_ROWS - 1) / TN_ROWS : 0;
    const uint32_t lds0 = lds_offset(lds);
    char *const lds_bytes = reinterpret_cast<char *>(lds);

    // copies of the stage of rows mt .. mt+31 into slot `slot`; rows past the end repeat the last one
    auto copy_stage = [&](int mt, int slot) __attribute__((always_inline)) {
        const int last = m_end - 1 - mt;
        const uint32_t to = lds0 + slot * STAGE;
        const char *y = reinterpret_cast<const char *>(p.dy + (size_t)mt * p.N1 + y0);
        const char *x = p.xbase(mt);
#pragma unroll
        for (int i = 0; i < Y_COPIES; ++i) {
            const int at = wave * Y_COPIES + i, w = at * 64 + lane, r = w / YC, c = (w % YC) ^ tn_swizzle<YB>(r);
            copy_to_lds(y, (uint32_t)(min(r, last) * p.N1 * 2 + c * 16), to + at * 1024);
        }
#pragma unroll
        for (int i = 0; i < X_COPIES; ++i) {
            const int at = wave * X_COPIES + i, w = at * 64 + lane, r = w / XC, c = (w % XC) ^ tn_swizzle<XB>(r);
            copy_to_lds(x, p.xoff(min(r, last), x0 + c * 8), to + Y_BYTES + at * 1024);
        }
    };

    f32x16 acc[TY][TX];
#pragma unroll
    for (int a = 0; a < TY; ++a)
#pragma unroll
        for (int b = 0; b < TX; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    // bias gradient (column sums of dY), kept by the workgroups of the first tile column: a thread takes the same eight
    // dY columns of every stage (256 is a multiple of YC) and adds them in fp32
    float bs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bool keeps_bias = bx == 0;

#pragma unroll
    for (int s = 0; s < RING - 1; ++s)
        if (s < stages) copy_stage(m_begin + s * TN_ROWS, s);
    int slot = 0;
    for (int s = 0; s < stages; ++s) {
        // stage s has arrived when only the copies of the stages issued after it are outstanding
        const int after = min(stages - 1 - s, RING - 2);
        if (after >= 3) wait_vmem<(RING > 4 ? 3 : 0) * COPIES>();
        else if (after == 2) wait_vmem<(RING > 3 ? 2 : 0) * COPIES>();
        else if (after == 1) wait_vmem<COPIES>();
        else wait_vmem<0>();
        __syncthreads();
        const int mt = m_begin + s * TN_ROWS;
        // everyone has read the stage before: its slot takes the next copies
        if (s + RING - 1 < stages) copy_stage(mt + (RING - 1) * TN_ROWS, slot == 0 ? RING - 1 : slot - 1);
        char *const sY = lds_bytes + slot * STAGE, *const sX = sY + Y_BYTES;
        if (mt + TN_ROWS > m_end) {                              // the last stage: rows past the end are zero
            for (int w = (m_end - mt) * YC + tid; w < TN_ROWS * YC; w += 256) reinterpret_cast<u32x4 *>(sY)[w] = zero_u4();
            for (int w = (m_end - mt) * XC + tid; w < TN_ROWS * XC; w += 256) reinterpret_cast<u32x4 *>(sX)[w] = zero_u4();
            __syncthreads();
        }
#pragma unroll
        for (int kk = 0; kk < TN_ROWS / 16; ++kk) {
            bf16x8 fy[TY], fx[TX];
#pragma unroll
            for (int a = 0; a < TY; ++a) fy[a] = tr_fragment<YB>(sY, kk * 16, (wy * TY + a) * 32, lane);
#pragma unroll
            for (int b = 0; b < TX; ++b) fx[b] = tr_fragment<XB>(sX, kk * 16, (wx * TX + b) * 32, lane);
#pragma unroll
            for (int a = 0; a < TY; ++a)
#pragma unroll
                for (int b = 0; b < TX; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fy[a], fx[b], acc[a][b], 0, 0, 0);
        }
        if (keeps_bias) {
#pragma unroll
            for (int i = 0; i < TN_ROWS * YC / 256; ++i) {
                const int w = tid + 256 * i, r = w / YC;
                const bf16x8 f = as_bf16x8(reinterpret_cast<const u32x4 *>(sY)[w ^ tn_swizzle<YB>(r)]);
#pragma unroll
                for (int e = 0; e < 8; ++e) bs[e] += (float)f[e];
            }
        }
        slot = slot == RING - 1 ? 0 : slot + 1;
    }

    float *out = part + (size_t)split * ((size_t)p.N1 * p.KP + p.N1);
    const int fr = lane & 31, fg = lane >> 5;
#pragma unroll
    for (int a = 0; a < TY; ++a)
#pragma unroll
        for (int b = 0; b < TX; ++b) {
            const int k = x0 + (wx * TX + b) * 32 + fr;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int n = y0 + (wy * TY + a) * 32 + 8 * (r >> 2) + 4 * fg + (r & 3);
                out[(size_t)n * p.KP + k] = acc[a][b][r];
            }
        }
    if (keeps_bias) {
        // the 256/YC threads that share a column add their sums in thread order
        __syncthreads();
        float *scr = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int e = 0; e < 8; ++e) scr[(tid / YC) * BN1 + (tid % YC) * 8 + e] = bs[e];
        __syncthreads();
        if (tid < BN1) {
            float t = scr[tid];
            for (int g = 1; g < 256 / YC; ++g) t += scr[g * BN1 + tid];
            out[(size_t)p.N1 * p.KP + y0 + tid] = t;
        }
    }
}

}  // namespace arn
