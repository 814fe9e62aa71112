// Parameter update rules on the flat fp32 vector (appendix "Update Rule for Multi-Step Asynchronous Adam";
// RMSProp as named in appendix "Experiment Details"), and the single-launch conversion of the flat
// parameters into every packed layout the network kernels read.
//
// The update kernels are elementwise and HBM-bound: every thread owns four consecutive parameters and moves
// each state array with one 16-byte load and one 16-byte store.  All arithmetic is fp32; scalars that
// depend on the step count (the bias-correction factor a, beta^n of a merge) are formed on the host in
// fp64 and passed in.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "arn_gemm.h"
#include "arn_layout.h"
#include "arn_small_kernels.h"

namespace arn {

typedef float f32x4u __attribute__((ext_vector_type(4)));

enum { RULE_RMSPROP = 0, RULE_ADAM = 1, RULE_ADAM_LOCAL = 2, RULE_MERGE = 3 };

struct UpdateArgs {
    float *theta, *m, *v;          // RMSProp: v = accumulator of squared gradients, m unused
    const float *g;
    float *a_g, *a_g2, *a_s;       // local accumulators (RULE_ADAM_LOCAL, RULE_MERGE)
    float *theta_c, *m_c, *v_c;    // central values (RULE_MERGE)
    long n;
    float a;                       // RMSProp: learning rate; Adam: r*sqrt(1-beta2^t)/(1-beta1^t)
    float beta1, beta2;            // RMSProp: beta2 = rho.  RULE_MERGE: coefficients (1-beta1), (1-beta2) use these
    float eps;
    float beta1_n, beta2_n;        // RULE_MERGE: beta^n
};

// One element of a rule.  State goes in and out through references.  Fused products are written out, so that every kernel
// that applies a rule rounds alike (the compiler chooses per context which product of a sum to fuse).
template <int RULE>
struct Elem {
    static __device__ __forceinline__ void apply(const UpdateArgs &p, float &th, float &m, float &v, float g,
                                                  float &ag, float &ag2, float &as) {
        if constexpr (RULE == RULE_RMSPROP) {
            v = fmaf(p.beta2, v, (1.f - p.beta2) * g * g);
            th = th - p.a * g / sqrtf(v + p.eps);
        } else if constexpr (RULE == RULE_MERGE) {
            // merge of one learner's accumulated steps into the central values (third block of equations of the appendix)
            th = th - as;
            m = fmaf(p.beta1_n, m, (1.f - p.beta1) * ag);
            v = fmaf(p.beta2_n, v, (1.f - p.beta2) * ag2);
            ag = ag2 = as = 0.f;
        } else {
            m = fmaf(p.beta1, m, (1.f - p.beta1) * g);
            v = fmaf(p.beta2, v, (1.f - p.beta2) * g * g);
            const float s = p.a * m / (sqrtf(v) + p.eps);
            th = th - s;
            if constexpr (RULE == RULE_ADAM_LOCAL) {
                ag = fmaf(p.beta1, ag, g);
                ag2 = fmaf(p.beta2, ag2, g * g);
                as = as + s;
            }
        }
    }
};

// The state of a rule at one parameter (V = float) or at four consecutive ones (V = a vector of four).  A merge reads the
// central values and writes them to the local copies too.
__device__ __forceinline__ float lane_of(float v, int) { return v; }
__device__ __forceinline__ void set_lane(float &v, int, float x) { v = x; }
template <class V> __device__ __forceinline__ float lane_of(const V &v, int e) { return v[e]; }
template <class V> __device__ __forceinline__ void set_lane(V &v, int e, float x) { v[e] = x; }
template <int RULE, class V>
struct RuleState {
    static constexpr bool MOMENT = RULE != RULE_RMSPROP, ACCU = RULE == RULE_ADAM_LOCAL || RULE == RULE_MERGE;
    static constexpr bool CENTRAL = RULE == RULE_MERGE;
    V th, m, v, g, ag, ag2, as;
    static __device__ __forceinline__ V get(const float *a, long i) { return *(const V *)(a + i); }
    static __device__ __forceinline__ void put(float *a, long i, const V &x) { *(V *)(a + i) = x; }
    __device__ __forceinline__ void load(const UpdateArgs &p, long i) {
        th = get(CENTRAL ? p.theta_c : p.theta, i);
        v = get(CENTRAL ? p.v_c : p.v, i);
        m = g = ag = ag2 = as = V{};
        if constexpr (!CENTRAL) g = get(p.g, i);
        if constexpr (MOMENT) m = get(CENTRAL ? p.m_c : p.m, i);
        if constexpr (ACCU) { ag = get(p.a_g, i); ag2 = get(p.a_g2, i); as = get(p.a_s, i); }
    }
    __device__ __forceinline__ void step_and_store(const UpdateArgs &p, long i) {
#pragma unroll
        for (int e = 0; e < (int)(sizeof(V) / 4); ++e) {
            float t = lane_of(th, e), mm = lane_of(m, e), vv = lane_of(v, e);
            float x = lane_of(ag, e), y = lane_of(ag2, e), z = lane_of(as, e);
            Elem<RULE>::apply(p, t, mm, vv, lane_of(g, e), x, y, z);
            set_lane(th, e, t); set_lane(m, e, mm); set_lane(v, e, vv);
            set_lane(ag, e, x); set_lane(ag2, e, y); set_lane(as, e, z);
        }
        if constexpr (CENTRAL) { put(p.theta_c, i, th); put(p.m_c, i, m); put(p.v_c, i, v); }
        put(p.theta, i, th);
        put(p.v, i, v);
        if constexpr (MOMENT) put(p.m, i, m);
        if constexpr (ACCU) { put(p.a_g, i, ag); put(p.a_g2, i, ag2); put(p.a_s, i, as); }
    }
};

template <int RULE>
__global__ __launch_bounds__(256) void update_kernel(UpdateArgs p) {
    const long i0 = ((long)blockIdx.x * 256 + threadIdx.x) * 4;   // four parameters
    if (i0 + 4 <= p.n) {
        RuleState<RULE, f32x4u> x;
        x.load(p, i0);
        x.step_and_store(p, i0);
        return;
    }
    for (long i = i0; i < p.n; ++i) {
        RuleState<RULE, float> x;
        x.load(p, i);
        x.step_and_store(p, i);
    }
}

// ------------------------- all packed layouts in one launch -------------------------
// The packed blob has 14 regions (five forward weight matrices with their lo parts, five bias vectors,
// four input-gradient layouts).  One launch covers them all: a block finds the region its index falls in
// (uniform per block) and applies that region's index map.
enum {
    PK_W1 = 0, PK_W2, PK_W3, PK_WFC, PK_WH, PK_B1, PK_B2, PK_B3, PK_BFC, PK_BH, PK_WHD, PK_WFCD, PK_W3D, PK_W2D,
    PK_COUNT
};
struct PackSeg {
    int first_block;
    long n;
    void *out, *out_lo;
    void *out_f16;     // fp16 copy of a forward layout, or null
};
// The fc matrix (95 % of the parameters) is laid out by tile blocks instead: elementwise maps would read it with
// a stride of one row (input-gradient layout) or of P3 floats (forward layout).  A tile is PACK_FC_ROWS hidden
// units x PACK_FC_CH conv3 channels x all P3 positions -- contiguous runs of PACK_FC_CH * P3 floats in the flat
// vector -- staged in LDS and written out as 16-byte words of eight channels (forward layout, hi and lo) and of
// eight hidden units (input-gradient layout).  Eight rows per tile measured best (12.2 us for the whole launch
// against 13.1 with sixteen and 16 with thirty-two; the elementwise maps took 18.3).
constexpr int PACK_FC_ROWS = 8, PACK_FC_CH = 8;
// fp16 copy of a weight: values beyond the largest half are clamped to it instead of becoming infinite
__device__ __forceinline__ _Float16 to_f16_finite(float v) { return (_Float16)fminf(fmaxf(v, -65504.f), 65504.f); }
constexpr int PACK_FC_MAX_P3 = 108;   // 12 x 9 positions after conv3 on 104 x 80 frames
// LDS row: 8 modulo 64 words, so that eight rows x eight neighbouring positions are 64 different banks
constexpr int PACK_FC_LDS_ROW = PACK_FC_CH * PACK_FC_MAX_P3 + 8;
static_assert(P3 <= PACK_FC_MAX_P3 && GeoPaper::P3 <= PACK_FC_MAX_P3, "fc tile buffer");
static_assert(PACK_FC_CH == 8 && PACK_FC_ROWS % 8 == 0, "fc tile shape");
typedef float PackTile[PACK_FC_ROWS][PACK_FC_LDS_ROW];
template <class G>
struct PackPlan {
    PackSeg seg[PK_COUNT];
    int fc_first_block;                      // blocks from here on are fc tiles
    __bf16 *fc_hi, *fc_lo, *fc_dgrad;
    _Float16 *fc_f16;
    long w1, w2, w3, wfc, b1, b2, b3, bfc;   // offsets in the flat vector
    MapHeadRow<G::NHID> hr;
    int NHP;
    int blocks;
};

template <class G>
inline PackPlan<G> make_pack_plan(const Dims &d, void *w_packed) {
    const ParamOffsets po = param_offsets(d);
    const PackedOffsets o = packed_offsets(d);
    char *b = (char *)w_packed;
    PackPlan<G> pl;
    pl.w1 = (long)po.w1; pl.w2 = (long)po.w2; pl.w3 = (long)po.w3; pl.wfc = (long)po.wfc;
    pl.b1 = (long)po.b1; pl.b2 = (long)po.b2; pl.b3 = (long)po.b3; pl.bfc = (long)po.bfc;
    pl.hr = head_rows<G::NHID>(d, po);
    pl.NHP = d.NHP;
    auto set = [&](int k, long n, size_t out, size_t lo, bool has_lo) {
        pl.seg[k].n = n;
        pl.seg[k].out = b + out;
        pl.seg[k].out_lo = has_lo ? b + lo : nullptr;
        pl.seg[k].out_f16 = nullptr;
    };
    set(PK_W1, (long)G::NC1 * KW1, o.w1, o.w1l, true);
    set(PK_W2, (long)G::NC2 * G::KW2, o.w2, o.w2l, true);
    set(PK_W3, (long)d.c3 * KW3, o.w3, o.w3l, true);
    set(PK_WFC, 0, o.wfc, o.wfcl, true);          // by tile blocks, below
    set(PK_WH, (long)d.NHP * G::NHID, o.wh, o.whl, true);
    set(PK_B1, G::NC1, o.b1, 0, false);
    set(PK_B2, G::NC2, o.b2, 0, false);
    set(PK_B3, d.c3, o.b3, 0, false);
    set(PK_BFC, G::NHID, o.bfc, 0, false);
    set(PK_BH, d.NHP, o.bh, 0, false);
    set(PK_WHD, (long)G::NHID * d.NHP, o.whd, 0, false);
    set(PK_WFCD, 0, o.wfcd, 0, false);            // by tile blocks, below
    pl.seg[PK_W1].out_f16 = b + o.w1h; pl.seg[PK_W2].out_f16 = b + o.w2h; pl.seg[PK_W3].out_f16 = b + o.w3h;
    pl.fc_hi = (__bf16 *)(b + o.wfc); pl.fc_lo = (__bf16 *)(b + o.wfcl); pl.fc_dgrad = (__bf16 *)(b + o.wfcd);
    pl.fc_f16 = (_Float16 *)(b + o.wfch);
    set(PK_W3D, (long)d.c3 * KW3, o.w3d, 0, false);
    set(PK_W2D, (long)4 * G::NC1 * 4 * G::NC2, o.w2d, 0, false);
    int blk = 0;
    for (int k = 0; k < PK_COUNT; ++k) {
        pl.seg[k].first_block = blk;
        blk += (int)((pl.seg[k].n + 255) / 256);
    }
    pl.fc_first_block = blk;
    pl.blocks = blk + (G::NHID / PACK_FC_ROWS) * (G::NCL / PACK_FC_CH);
    return pl;
}

// One fc tile: hidden units n0 .. n0 + PACK_FC_ROWS - 1, channels c0 .. c0 + PACK_FC_CH - 1.
// Flat order Wfc[n][c * P + pos]; forward layout [n][pos * NC + c]; input-gradient layout [pos * NC + c][n].
template <class G>
struct PackFcTile {
    static constexpr int RUN = PACK_FC_CH * G::PL, CT = G::NCL / PACK_FC_CH;   // floats per hidden unit; tiles per hidden unit
    static_assert(G::NHID % PACK_FC_ROWS == 0 && G::NCL % PACK_FC_CH == 0 && G::PL <= PACK_FC_MAX_P3, "fc tile shape");
    int n0, c0;
    __device__ __forceinline__ explicit PackFcTile(int tile) : n0(tile / CT * PACK_FC_ROWS), c0(tile % CT * PACK_FC_CH) {}
    // offset in the matrix of float e of row r
    __device__ __forceinline__ long at(int r, int e) const { return (long)(n0 + r) * G::FEAT + (long)c0 * G::PL + e; }
};
template <class G>
__device__ __forceinline__ void pack_fc_read(const PackPlan<G> &pl, const float *__restrict__ w, PackFcTile<G> f, PackTile &s_t) {
    constexpr int run = PackFcTile<G>::RUN, NL = (PACK_FC_ROWS * run + 255) / 256;
    const int tid = threadIdx.x;
    float v_in[NL];   // all loads of the tile in flight before the first is used
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        int i = tid + 256 * j;
        i = i < PACK_FC_ROWS * run ? i : PACK_FC_ROWS * run - 1;
        v_in[j] = w[pl.wfc + f.at(i / run, i % run)];
    }
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int i = tid + 256 * j;
        if (i < PACK_FC_ROWS * run) s_t[i / run][i % run] = v_in[j];
    }
}
template <class G>
__device__ __forceinline__ void pack_fc_write(const PackPlan<G> &pl, PackFcTile<G> f, const PackTile &s_t) {
    constexpr int p3 = G::PL, NC = G::NCL, feat = G::FEAT, run = PackFcTile<G>::RUN;
    const int n0 = f.n0, c0 = f.c0, tid = threadIdx.x;
    // forward layout: one 16-byte word = channels c0 .. c0+7 of (row r, position pos)
    // (fragment order, frag_index: the eight rows' words are neighbours)
    for (int i = tid; i < PACK_FC_ROWS * p3; i += 256) {
        const int r = i % PACK_FC_ROWS, pos = i / PACK_FC_ROWS;
        float v[PACK_FC_CH];
#pragma unroll
        for (int c = 0; c < PACK_FC_CH; ++c) v[c] = s_t[r][c * p3 + pos];
        bf16x8 hi, lo;
        f16x8 hf;
#pragma unroll
        for (int c = 0; c < PACK_FC_CH; ++c) {
            hi[c] = (__bf16)v[c];
            lo[c] = (__bf16)(v[c] - (float)hi[c]);
            hf[c] = to_f16_finite(v[c]);
        }
        const size_t at = (size_t)frag_index(n0 + r, (long)pos * NC + c0, feat);
        *reinterpret_cast<bf16x8 *>(pl.fc_hi + at) = hi;
        *reinterpret_cast<bf16x8 *>(pl.fc_lo + at) = lo;
        *reinterpret_cast<f16x8 *>(pl.fc_f16 + at) = hf;
    }
    // input-gradient layout: one 16-byte word = hidden units n0 + 8h .. + 7 of (position pos, channel c)  (h = 0 with eight rows)
    for (int i = tid; i < (PACK_FC_ROWS / 8) * run; i += 256) {
        const int h = i / run, e = i - h * run, c = e / p3, pos = e - c * p3;
        bf16x8 hi;
#pragma unroll
        for (int r = 0; r < 8; ++r) hi[r] = (__bf16)s_t[8 * h + r][e];
        *reinterpret_cast<bf16x8 *>(pl.fc_dgrad + frag_index((long)pos * NC + c0 + c, n0 + 8 * h, G::NHID)) = hi;
    }
}

template <class G>
__global__ __launch_bounds__(256) void pack_all_kernel(const PackPlan<G> pl, const float *__restrict__ w) {
    if ((int)blockIdx.x >= pl.fc_first_block) {
        __shared__ PackTile s_t;
        const PackFcTile<G> f((int)blockIdx.x - pl.fc_first_block);
        pack_fc_read<G>(pl, w, f, s_t);
        __syncthreads();
        pack_fc_write<G>(pl, f, s_t);
        return;
    }
    int k = 0;
#pragma unroll
    for (int j = 1; j < PK_COUNT; ++j) k = (int)blockIdx.x >= pl.seg[j].first_block ? j : k;
    // region fields selected without dynamic indexing of the argument block
    int first = 0;
    long n = 0;
    void *out = nullptr, *out_lo = nullptr, *out_f16 = nullptr;
#pragma unroll
    for (int j = 0; j < PK_COUNT; ++j)
        if (j == k) { first = pl.seg[j].first_block; n = pl.seg[j].n; out = pl.seg[j].out; out_lo = pl.seg[j].out_lo; out_f16 = pl.seg[j].out_f16; }
    const long i = (long)((int)blockIdx.x - first) * 256 + threadIdx.x;
    if (i >= n) return;
    long s;
    switch (k) {
    case PK_W1: s = pl.w1 + i; break;
    case PK_W2: s = MapConvFwd<G::NC1, K2>{pl.w2}(i); break;
    case PK_W3: s = MapConvFwd<C2, K3>{pl.w3}(i); break;
    case PK_WH: s = MapHeadFwd<G::NHID>{pl.hr}(i); break;
    case PK_B1: s = pl.b1 + i; break;
    case PK_B2: s = pl.b2 + i; break;
    case PK_B3: s = pl.b3 + i; break;
    case PK_BFC: s = pl.bfc + i; break;
    case PK_BH: s = MapHeadBias<G::NHID>{pl.hr}(i); break;
    case PK_WHD: s = MapHeadDgrad<G::NHID>{pl.hr, pl.NHP}(i); break;
    case PK_W3D: s = MapConv3Dgrad{pl.w3}(i); break;
    default: s = MapConv2Dgrad<G::NC1, G::NC2>{pl.w2}(i); break;
    }
    const float v = s >= 0 ? w[s] : 0.f;
    if (k >= PK_B1 && k <= PK_BH) {
        ((float *)out)[i] = v;
    } else {
        // every matrix is packed in fragment order (frag_index)
        long o = i;
        if (k == PK_W1) o = frag_index(i / KW1, i % KW1, KW1);
        else if (k == PK_W2) o = frag_index(i / G::KW2, i % G::KW2, G::KW2);
        else if (k == PK_W3 || k == PK_W3D) o = frag_index(i / KW3, i % KW3, KW3);
        else if (k == PK_W2D) o = frag_index(i / (4 * G::NC2), i % (4 * G::NC2), 4 * G::NC2);
        else if (k == PK_WH) o = frag_index(i / G::NHID, i % G::NHID, G::NHID);
        else if (k == PK_WHD) o = frag_index(i / pl.NHP, i % pl.NHP, pl.NHP);
        const __bf16 hi = (__bf16)v;
        ((__bf16 *)out)[o] = hi;
        if (out_lo) ((__bf16 *)out_lo)[o] = (__bf16)(v - (float)hi);
        if (out_f16) ((_Float16 *)out_f16)[o] = to_f16_finite(v);
    }
}

// ------------------------- a rule and every packed layout in one launch -------------------------
// An update with a re-pack: whoever updates a parameter also writes its packed copies, so the new values are not read back
// and there is one launch instead of two (a boundary costs about 4 us here, the read of theta 2).  Three ranges of
// workgroups: fc tiles as above; eight head rows each (through LDS: the forward layouts want eight neighbouring inputs in a
// 16-byte word, the input-gradient layout eight neighbouring rows); the convolutions and the fc bias, one parameter a thread.
// Bound by HBM: 28 bytes of state a parameter with Adam and 8 bytes of packed copies.  Adam on the categorical network (2.2 M
// parameters): 14.5 us, 4.5 TB/s of state, against 23.2 for rule and re-pack as two launches.
constexpr int PACK_HEAD_ROWS = PACK_FC_ROWS;
typedef float f32x4p __attribute__((ext_vector_type(4), aligned(4)));   // the value row starts at any parameter
template <class G>
inline int update_pack_blocks(const PackPlan<G> &pl) {
    return G::NHID / PACK_FC_ROWS * PackFcTile<G>::CT + pl.NHP / PACK_HEAD_ROWS + (int)((pl.wfc + G::NHID + 255) / 256);
}

// The packed copies of parameter i of the convolutions and the fc bias, the inverse of the Map* structs.
template <class G>
__device__ __forceinline__ void scatter_packed(const PackPlan<G> &pl, long i, float v) {
    auto matrix = [&](int seg, long at) {
        const __bf16 hi = (__bf16)v;
        ((__bf16 *)pl.seg[seg].out)[at] = hi;
        if (pl.seg[seg].out_lo) ((__bf16 *)pl.seg[seg].out_lo)[at] = (__bf16)(v - (float)hi);
        if (pl.seg[seg].out_f16) ((_Float16 *)pl.seg[seg].out_f16)[at] = to_f16_finite(v);
    };
    if (i >= pl.bfc) { ((float *)pl.seg[PK_BFC].out)[i - pl.bfc] = v; return; }
    if constexpr (G::HAS3) {
        if (i >= pl.b3) { ((float *)pl.seg[PK_B3].out)[i - pl.b3] = v; return; }
        if (i >= pl.w3) {
            const int e = (int)(i - pl.w3), co = e / KW3, ci = e % KW3 / (K3 * K3), ky = e % (K3 * K3) / K3, kx = e % K3;
            matrix(PK_W3, frag_index(co, (ky * K3 + kx) * C2 + ci, KW3));
            matrix(PK_W3D, frag_index(ci, ((K3 - 1 - ky) * K3 + K3 - 1 - kx) * 64 + co, KW3));
            return;
        }
    }
    if (i >= pl.b2) { ((float *)pl.seg[PK_B2].out)[i - pl.b2] = v; return; }
    if (i >= pl.w2) {
        const int e = (int)(i - pl.w2), co = e / G::KW2, ci = e % G::KW2 / (K2 * K2), ky = e % (K2 * K2) / K2, kx = e % K2;
        const int z = (ky & 1) * 2 + (kx & 1), tap = (1 - (ky >> 1)) * 2 + 1 - (kx >> 1);
        matrix(PK_W2, frag_index(co, (ky * K2 + kx) * G::NC1 + ci, G::KW2));
        matrix(PK_W2D, frag_index(z * G::NC1 + ci, tap * G::NC2 + co, 4 * G::NC2));
        return;
    }
    if (i >= pl.b1) { ((float *)pl.seg[PK_B1].out)[i - pl.b1] = v; return; }
    matrix(PK_W1, frag_index(i / KW1, i % KW1, KW1));
}

template <int RULE, class G>
__global__ __launch_bounds__(256) void update_pack_kernel(const PackPlan<G> pl, const UpdateArgs p) {
    __shared__ alignas(16) PackTile s_t;
    constexpr int AHEAD = RuleState<RULE, float>::ACCU ? 2 : 4;   // groups whose loads are in flight: 16 or 12 to 14 registers each
    const int tid = threadIdx.x;
    int b = blockIdx.x;
    constexpr int FC_TILES = G::NHID / PACK_FC_ROWS * PackFcTile<G>::CT;
    if (b < FC_TILES) {
        const PackFcTile<G> f(b);
        constexpr int R4 = PackFcTile<G>::RUN / 4, N4 = PACK_FC_ROWS * R4;   // groups of four parameters
        static_assert(PackFcTile<G>::RUN % 4 == 0 && G::FEAT % 4 == 0 && PACK_FC_LDS_ROW % 4 == 0, "16-byte groups");
#pragma unroll
        for (int j0 = 0; j0 * 256 < N4; j0 += AHEAD) {
            RuleState<RULE, f32x4u> x[AHEAD];
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) {
                const int q = tid + 256 * (j0 + j);
                if (q < N4) x[j].load(p, pl.wfc + f.at(q / R4, 4 * (q % R4)));
            }
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) {
                const int q = tid + 256 * (j0 + j);
                if (q >= N4) continue;
                x[j].step_and_store(p, pl.wfc + f.at(q / R4, 4 * (q % R4)));
                *(f32x4u *)&s_t[q / R4][4 * (q % R4)] = x[j].th;
            }
        }
        __syncthreads();
        pack_fc_write<G>(pl, f, s_t);
        return;
    }
    b -= FC_TILES;
    if (b < pl.NHP / PACK_HEAD_ROWS) {
        constexpr int R4 = G::NHID / 4, N4 = PACK_HEAD_ROWS * R4;
        static_assert(N4 % 256 == 0 && G::NHID <= PACK_FC_LDS_ROW, "head tile shape");
        const int r0 = b * PACK_HEAD_ROWS;
#pragma unroll
        for (int j = 0; j < N4 / 256; ++j) {
            const int q = tid + 256 * j, r = q / R4, e = 4 * (q % R4);
            const long row = pl.hr.wrow(r0 + r);
            f32x4u th = 0.f;     // rows past the last are zeros in the packed matrix
            if (row >= 0) {
                RuleState<RULE, f32x4p> x;
                x.load(p, row + e);
                x.step_and_store(p, row + e);
                th = x.th;
            }
            *(f32x4u *)&s_t[r][e] = th;
        }
        if (tid < PACK_HEAD_ROWS) {
            const long at = pl.hr.brow(r0 + tid);
            RuleState<RULE, float> x;
            x.th = 0.f;
            if (at >= 0) {
                x.load(p, at);
                x.step_and_store(p, at);
            }
            ((float *)pl.seg[PK_BH].out)[r0 + tid] = x.th;
        }
        __syncthreads();
        for (int i = tid; i < PACK_HEAD_ROWS * (G::NHID / 8); i += 256) {
            const int r = i % PACK_HEAD_ROWS, k = i / PACK_HEAD_ROWS * 8;
            bf16x8 hi, lo;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float v = s_t[r][k + c];
                hi[c] = (__bf16)v;
                lo[c] = (__bf16)(v - (float)hi[c]);
            }
            const long at = frag_index(r0 + r, k, G::NHID);
            *reinterpret_cast<bf16x8 *>((__bf16 *)pl.seg[PK_WH].out + at) = hi;
            *reinterpret_cast<bf16x8 *>((__bf16 *)pl.seg[PK_WH].out_lo + at) = lo;
        }
        for (int k = tid; k < G::NHID; k += 256) {
            bf16x8 hi;
#pragma unroll
            for (int r = 0; r < 8; ++r) hi[r] = (__bf16)s_t[r][k];
            *reinterpret_cast<bf16x8 *>((__bf16 *)pl.seg[PK_WHD].out + frag_index(k, r0, pl.NHP)) = hi;
        }
        return;
    }
    b -= pl.NHP / PACK_HEAD_ROWS;
    long i = (long)b * 256 + tid;
    if (i >= pl.wfc + G::NHID) return;
    if (i >= pl.wfc) i += pl.bfc - pl.wfc;
    RuleState<RULE, float> x;
    x.load(p, i);
    x.step_and_store(p, i);
    scatter_packed<G>(pl, i, x.th);
}

}  // namespace arn
