// Shapes of the Nature CNN, the packed-weight blob and the workspace carve-up.
// Host-side arithmetic only; shared by the API layer and the kernel launchers.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/arn.h"

namespace arn {

// network geometry (appendix "Atari Frame Processing": the standard
// 3-convolutional-layer network; 84x84 frames, no padding)
constexpr int IN_C = 4, IN_H = 84, IN_W = 84;
constexpr int OBS_BYTES = IN_C * IN_H * IN_W;            // 28224
constexpr int C1 = 32, K1 = 8, S1 = 4, H1 = 20;          // conv1 out 20x20
constexpr int C2 = 64, K2 = 4, S2 = 2, H2 = 9;           // conv2 out 9x9
constexpr int C3 = 64, K3 = 3, S3 = 1, H3 = 7;           // conv3 out 7x7
constexpr int P1 = H1 * H1, P2 = H2 * H2, P3 = H3 * H3;  // 400, 81, 49
constexpr int KW1 = IN_C * K1 * K1;                      // 256
constexpr int KW2 = C1 * K2 * K2;                        // 512
constexpr int KW3 = C2 * K3 * K3;                        // 576
constexpr int FEAT = C3 * P3;                            // 3136
constexpr int HID = 512;

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Frame size, padding and channel counts of the network as compile-time constants (the filter sizes and strides
// above are common to all).  Geo84 restates the constants above; GeoPaper is the appendix's own setting: 104x80
// frames, no padding on conv1, padding 1 on conv2 and conv3.  HL x WL: the last feature map, NCL its channels.
template <int IN_H_, int IN_W_, int PAD2_, int PAD3_, int NC1_ = arn::C1, int NC2_ = arn::C2, bool HAS3_ = true, int NHID_ = HID>
struct Geometry {
    static constexpr int IN_H = IN_H_, IN_W = IN_W_, PAD2 = PAD2_, PAD3 = PAD3_;
    static constexpr int NC1 = NC1_, NC2 = NC2_, NHID = NHID_, KW2 = NC1_ * K2 * K2;
    static constexpr bool HAS3 = HAS3_;
    static constexpr int H1 = (IN_H - K1) / S1 + 1, W1 = (IN_W - K1) / S1 + 1;
    static constexpr int H2 = (H1 + 2 * PAD2 - K2) / S2 + 1, W2 = (W1 + 2 * PAD2 - K2) / S2 + 1;
    static constexpr int H3 = (H2 + 2 * PAD3 - K3) / S3 + 1, W3 = (W2 + 2 * PAD3 - K3) / S3 + 1;
    static constexpr int P1 = H1 * W1, P2 = H2 * W2, P3 = H3 * W3;
    static constexpr int HL = HAS3 ? H3 : H2, WL = HAS3 ? W3 : W2, PL = HL * WL, NCL = HAS3 ? C3 : NC2;
    static constexpr int OBS_BYTES = IN_C * IN_H * IN_W, FEAT = NCL * PL;
};
typedef Geometry<84, 84, 0, 0> Geo84;
typedef Geometry<104, 80, 1, 1> GeoPaper;
// the 2-convolution network of the same appendix: 16 and 32 filters, no third convolution, 256 hidden units
typedef Geometry<104, 80, 1, 1, 16, 32, false, 256> GeoA3c;
static_assert(Geo84::P1 == P1 && Geo84::P2 == P2 && Geo84::P3 == P3 && Geo84::FEAT == FEAT, "84x84 constants");
static_assert(GeoPaper::H1 == 25 && GeoPaper::W1 == 19 && GeoPaper::H2 == 12 && GeoPaper::W2 == 9 &&
              GeoPaper::H3 == 12 && GeoPaper::W3 == 9 && GeoPaper::FEAT == 6912, "appendix: 25x19 -> 12x9 -> 12x9");
static_assert(GeoA3c::PL == 108 && GeoA3c::FEAT == 3456, "appendix: 25x19 -> 12x9");

struct Dims {
    int A = 0, head = 0, atoms = 0;
    int NH = 0;    // real head rows: A+1 (PV, DUEL), A (Q) or A*atoms (C51)
    int NHP = 0;   // head rows padded to a multiple of 64 (MFMA k-tile of the head dgrad)
    bool small = false;   // at most 32 head rows: the fused head kernel follows the fc GEMM (PV, Q, DUEL)
    bool vrow = false;    // the row after the A action rows is a state value (PV, DUEL)
    bool qhead = false;   // the head outputs are action values (Q, DUEL)
    int geom = ARN_GEOM_84;
    // channels of the convolutions (c3 = 0: none), conv2's contraction length, hidden units
    int c1 = C1, c2 = C2, c3 = C3, kw2 = KW2, hid = HID;
    int p1 = P1, p2 = P2, pl = P3, feat = FEAT, obs_bytes = OBS_BYTES;   // positions per sample after conv1, conv2 and the last convolution, fc inputs, bytes per observation
    bool ok = false;
};

template <class G>
inline void set_geometry(Dims &d) {
    d.c1 = G::NC1; d.c2 = G::NC2; d.c3 = G::HAS3 ? C3 : 0; d.kw2 = G::KW2; d.hid = G::NHID;
    d.p1 = G::P1; d.p2 = G::P2; d.pl = G::PL; d.feat = G::FEAT; d.obs_bytes = G::OBS_BYTES;
}
inline Dims make_dims(const arn_config *c) {
    Dims d;
    if (!c) return d;
    d.A = c->num_actions;
    d.head = c->head_kind;
    d.geom = c->geometry;
    if (d.geom == ARN_GEOM_84) set_geometry<Geo84>(d);
    else if (d.geom == ARN_GEOM_PAPER) set_geometry<GeoPaper>(d);
    else if (d.geom == ARN_GEOM_A3C) set_geometry<GeoA3c>(d);
    else return d;
    if (d.head == ARN_HEAD_PV || d.head == ARN_HEAD_Q || d.head == ARN_HEAD_DUEL) {
        if (d.A < 1 || d.A > 31) return d;
        d.atoms = 1;
        d.small = true;
        d.vrow = d.head != ARN_HEAD_Q;
        d.qhead = d.head != ARN_HEAD_PV;
        d.NH = d.A + (d.vrow ? 1 : 0);
    } else if (d.head == ARN_HEAD_C51) {
        d.atoms = c->num_atoms;
        if (d.A < 1 || d.A > 18 || d.atoms < 2 || d.atoms > 64) return d;
        if (!(c->v_max > c->v_min)) return d;
        d.NH = d.A * d.atoms;
    } else {
        return d;
    }
    d.NHP = (int)align_up((size_t)d.NH, 64);
    d.ok = true;
    return d;
}

// offsets (in fp32 entries) into the canonical flat parameter vector
struct ParamOffsets {
    size_t w1, b1, w2, b2, w3, b3, wfc, bfc, wh, bh, wv, bv, total;
};
inline ParamOffsets param_offsets(const Dims &d) {
    ParamOffsets o{};
    size_t p = 0;
    o.w1 = p; p += (size_t)d.c1 * KW1;
    o.b1 = p; p += d.c1;
    o.w2 = p; p += (size_t)d.c2 * d.kw2;
    o.b2 = p; p += d.c2;
    o.w3 = p; p += (size_t)d.c3 * KW3;
    o.b3 = p; p += d.c3;
    o.wfc = p; p += (size_t)d.hid * d.feat;
    o.bfc = p; p += d.hid;
    if (d.vrow) {
        o.wh = p; p += (size_t)d.A * d.hid;
        o.bh = p; p += d.A;
        o.wv = p; p += d.hid;
        o.bv = p; p += 1;
    } else {
        o.wh = p; p += (size_t)d.NH * d.hid;
        o.bh = p; p += d.NH;
        o.wv = o.bv = p;
    }
    o.total = p;
    return o;
}

// byte offsets into the packed blob
struct PackedOffsets {
    size_t w1, w2, w3, wfc, wh;          // forward layouts  [N][K'] bf16 (high parts)
    size_t b1, b2, b3, bfc, bh;          // fp32 biases
    size_t w1l, w2l, w3l, wfcl, whl;     // low parts (w - hi) for the three-product inference path
    size_t whd, wfcd, w3d, w2d;          // input-gradient layouts
    size_t w1h, w2h, w3h, wfch;          // fp16 copies of the forward layouts (single-product, no-gradient forward)
    size_t total;
};
inline PackedOffsets packed_offsets(const Dims &d) {
    PackedOffsets o{};
    size_t p = 0;
    auto take = [&](size_t bytes) { size_t at = p; p = align_up(p + bytes, 256); return at; };
    const size_t w1 = (size_t)d.c1 * KW1 * 2, w2 = (size_t)d.c2 * d.kw2 * 2, w3 = (size_t)d.c3 * KW3 * 2;
    const size_t wfc = (size_t)d.hid * d.feat * 2, wh = (size_t)d.NHP * d.hid * 2;
    o.w1 = take(w1);
    o.w2 = take(w2);
    o.w3 = take(w3);
    o.wfc = take(wfc);
    o.wh = take(wh);
    o.b1 = take(d.c1 * 4);
    o.b2 = take(d.c2 * 4);
    o.b3 = take(d.c3 * 4);
    o.bfc = take(d.hid * 4);
    o.bh = take((size_t)d.NHP * 4);
    o.w1l = take(w1);
    o.w2l = take(w2);
    o.w3l = take(w3);
    o.wfcl = take(wfc);
    o.whl = take(wh);
    o.whd = take(wh);
    o.wfcd = take(wfc);
    o.w3d = take(w3);
    o.w2d = take((size_t)4 * d.c1 * 4 * d.c2 * 2);
    o.w1h = take(w1);
    o.w2h = take(w2);
    o.w3h = take(w3);
    o.wfch = take(wfc);
    o.total = p;
    return o;
}

// how many batch slices each weight-gradient GEMM is cut into (fixed function
// of B only, so the summation order -- and the bits of dW -- never change)
struct Splits {
    int c1, c2, c3, fc, hd;
};
inline int pick_split(long rows, int tiles, int target_wgs) {
    long iters = (rows + 63) / 64;
    long s = target_wgs / tiles;
    if (s < 1) s = 1;
    if (s > iters) s = iters;
    return (int)s;
}
constexpr int CONV3_WG_G = 4;   // samples staged per iteration by the conv3 weight-gradient kernel
template <class G>
struct Conv2WgradG {            // ... and by conv2's
    static constexpr int value = G::HAS3 ? 2 : 4;
};
inline int conv2_wg_g(const Dims &d) { return d.c3 ? Conv2WgradG<Geo84>::value : Conv2WgradG<GeoA3c>::value; }
// sample-resident weight-gradient kernels: samples per workgroup and number of workgroups
inline int resident_spw(int B, int target_wgs) { return (B + target_wgs - 1) / target_wgs; }
inline int resident_groups(int B, int target_wgs) {
    const int spw = resident_spw(B, target_wgs);
    return (B + spw - 1) / spw;
}
// The convolutions' backward (conv_backward_kernel): ranges of workgroups, one workgroup per CU, that share the 256 CUs in
// one round.  A range's workgroup count follows its measured time per sample (relative to the others), so that all finish
// together; every workgroup has a prologue of about 3 us and writes a full fp32 partial, so one round of longer workgroups
// also means less of both.  (256 workgroups for the first range and 256 for the others, in two rounds, took 61 + 14.5 us
// with the sums at 2048 samples and 84x84 frames, this 56.5 + 11; 104x80 frames: 122 against 75 us.)
// A range's time is first + cost per sample: on 84x84 frames the first range's workgroups take about 2 us longer before and after
// their samples than the others', and conv2's weight gradient, which reads the most bytes in a given time, costs more per sample in
// batches whose activations the 256 MB Infinity Cache does not hold (about 110 KB a sample: from 2400 samples on).  Launch and
// sums of the partials in us, with 3.2 : 1.5 : 1.25 and no first time / 3.2 : 1.7 : 1.05 and none / these, 150 samples: 20.1 / 23.2 /
// 20.1, 333: 28.2 / 27.0 / 26.2, 560: 30.2 / 32.8 / 30.2, 1000: 40.0 / 42.7 / 40.0, 1500: 51.0 / 52.5 / 51.2, 2048: 64.9 / 65.6 / 64.7, 2500:
// 82.4 / 81.1 / 79.0, 4096: 123.5 / 115.8 / 115.8.  Of 47 batches from 100 to 8192 none is more than 1.4% above the better of the other two.
// For the other networks no ratio tried near theirs was faster.
struct ConvBwdCost { float first, c1, c2, c3; };   // c1: conv2 input gradient with conv1 weight gradient, c2, c3: conv2's, conv3's weight gradient
inline ConvBwdCost conv_bwd_cost(int geom, int B) {
    if (geom == ARN_GEOM_84) return {2.f, 3.2f, B <= 2400 ? 1.5f : 1.7f, 1.05f};
    if (geom == ARN_GEOM_PAPER) return {0.f, 3.f, 1.5f, 1.5f};
    return {0.f, 3.5f, 1.f, 0.f};
}
struct ConvBwdSplit { int spw1, spw2, spw3; };   // samples per workgroup
// Workgroups of the first, of either other range, at most: the largest counts that the rule below comes to for any batch (204
// samples on the 2-convolution network; 337 samples on 104x80).  The reported workspace sizes rely on them.
constexpr int CONV_BWD_MOST1 = 204, CONV_BWD_MOST2 = 85;
inline ConvBwdSplit conv_bwd_split(const Dims &d, int B, int most1 = CONV_BWD_MOST1, int most2 = CONV_BWD_MOST2) {
    const ConvBwdCost c = conv_bwd_cost(d.geom, B);
    const int g2 = conv2_wg_g(d), g3 = CONV3_WG_G;
    ConvBwdSplit s;
    for (double t = (double)B * (c.c1 + c.c2 + c.c3) / 256;; t *= 1.01) {
        auto per = [&](double first, double cost, int g) { const int n = (int)((t - first) / (cost * g)); return (n < 1 ? 1 : n) * g; };
        s.spw1 = per(c.first, c.c1, 1);
        s.spw2 = per(0, c.c2, g2);
        s.spw3 = d.c3 ? per(0, c.c3, g3) : 1 << 30;
        const int n1 = (B + s.spw1 - 1) / s.spw1, n2 = (B + s.spw2 - 1) / s.spw2, n3 = d.c3 ? (B + s.spw3 - 1) / s.spw3 : 0;
        if (n1 + n2 + n3 <= 256 && n1 <= most1 && n2 <= most2 && n3 <= most2) return s;
    }
}
// Positions per workgroup tile of a dense contraction over M rows and N columns: 128 where that makes at least 256 workgroups,
// fewer (more workgroups) below.
inline int dense_tile(long M, int N) {
    const long nt = (N + 127) / 128;
    return (M + 127) / 128 * nt >= 256 ? 128 : (M + 63) / 64 * nt >= 256 ? 64 : 32;
}
// Hidden units per workgroup tile of the fc layer's weight gradient: 256 (64 x 64 outputs per wavefront, a third fewer LDS
// reads per product than 64 x 32, and half the act3 traffic, for twice the ranges of the batch and so twice the partials) for batches
// that have at least 500 tiles of 128 x 128 in the input gradient (84x84: 2433 samples, 104x80: 1153); with fewer, the launch is a few
// rounds of workgroups or less, and what the launch gains the sums of the partials lose.  Launch and sums in us, 128 / 256 units, 84x84:
// 333 samples 20.7 / 23.2, 2048: 39.8 / 38.5, 4096: 69.4 / 64.2, 8192: 118.4 / 104.5; 104x80, 512 samples: 31.5 / 34.0.  Whole A2C step,
// 84x84: 1281 samples 178.9 / 180.9, 1800: 228.3 / 230.9, 2048: 237.3 / 237.0, 2304: 268.6 / 267.6, 2432: 284.5 / 280.8, 4096: 419.5 / 414.7, 8192:
// 777.8 / 768.4; 104x80: 900 samples 198.6 / 204.4, 1100: 245.2 / 247.4, 1153: 247.0 / 247.6, 1408: 280.6 / 281.6, 1600: 312.3 / 310.3, 2048: 350.2 /
// 347.3.  By 84x84 alone the line would lie at 2049 samples, by 104x80 alone at about 1450, where they are level.
inline int fc_wgrad_units(int feat, int hid, int B) {
    return hid > 256 && (long)((B + 127) / 128) * ((feat + 127) / 128) >= 500 ? 256 : 128;
}
inline Splits make_splits(const Dims &d, int B) {
    Splits s;
    const ConvBwdSplit cs = conv_bwd_split(d, B);
    s.c1 = (B + cs.spw1 - 1) / cs.spw1;
    s.c2 = (B + cs.spw2 - 1) / cs.spw2;
    s.c3 = d.c3 ? (B + cs.spw3 - 1) / cs.spw3 : 0;
    // the dense layers' weight-gradient GEMMs are cut along the batch so that about 400 to 500 workgroups exist
    s.fc = pick_split(B, (d.feat / 64) * (d.hid / fc_wgrad_units(d.feat, d.hid, B)), d.geom == ARN_GEOM_84 ? 392 : 512);
    s.hd = pick_split(B, (d.hid / 128) * (d.NHP / 64), 256);
    return s;
}

// number of k ranges the fc forward GEMM is cut into (fills the chip when B/128 * 4 tiles are too few)
// f16: the one-product fc layer of the no-gradient forward, whose GEMM is a third of the work: at most eight ranges (the
// kernel also counts on at least eight stages of 32 in a range; the three-product layer on four).
// Small batches run in fc_small_kernel (one workgroup per 16 or 32 units and 16 or 32 samples, no k ranges in memory).  Its
// workgroups of one XCD share a band of weights and each XCD reads all activations, so it pays as long as those are few:
// up to about 2.5 M of them, counting hi and lo parts (one product, 3136 inputs, 256 samples: 10.8 us with the head
// against 8.4 + 5.7; three products, 6912 inputs, 512 samples: 29.6 against 18.8).
constexpr int FC_SMALL_MAX = 512;
inline bool fc_small(int feat, int B, bool f16) { return B <= FC_SMALL_MAX && (long)B * feat * (f16 ? 1 : 2) <= 2500000; }
// Tile of a workgroup: the smallest (most workgroups) that does not need more than 128 of them, at most 32 x 32.
struct FcTile { int units, rows; };
inline FcTile fc_small_tile(int hid, int B) {
    const int n = hid / 16;
    if (n * ((B + 15) / 16) <= 128) return {16, 16};
    if (n * ((B + 31) / 32) <= 128) return {16, 32};
    return {32, 32};
}
// Samples per workgroup tile of that GEMM: 128, or 64 where 128 would need more than eight ranges of the contraction to
// fill the chip: the partial sums are written and read back once per range (104x80, 512 samples: 64 takes the one-product
// layer from 13.7 to 10.5 us and the gradient step's layer and heads from 27.1 to 26.8).
inline int fc_tile(int hid, int B) { return ((B + 127) / 128) * (hid / 128) >= 32 ? 128 : 64; }
inline int fc_ksplit(int feat, int hid, int B, bool f16) {
    if (fc_small(feat, B, f16)) return 1;
    const int bm = fc_tile(hid, B);
    const int tiles = ((B + bm - 1) / bm) * (hid / 128);
    int ks = 256 / tiles;
    if (ks < 1) ks = 1;
    const int cap = f16 ? 8 : 16;   // the consumer adds the ranges one after the other: more of them costs it more than the GEMM gains
    if (ks > cap) ks = cap;
    return ks;
}

// Samples per workgroup of the fused policy/value head kernel in the gradient step (at most 16): eight keep all
// CUs busy at a few thousand samples; above that sixteen fill the MFMA's 16 sample columns and halve the workgroups;
// small batches are spread over more CUs, four samples each (one CU's L1 rate bounds the addition of the fc partials).
inline int loss_block(int B) { return B >= 4096 ? 16 : B <= 512 ? 4 : 8; }
constexpr int C51_WAVES = 4;      // wavefronts per block in the C51 kernels (one sample per wavefront at a time)
// Samples each wavefront of c51_loss_kernel takes one after the other: a block also writes one fp32 partial of the
// head's bias gradient, so large batches use fewer, longer blocks.
inline int c51_loss_spw(int B) { return B <= 2048 ? 1 : 4; }

// bytes of one sample's sign bits of act1, in whole 4-byte words
constexpr int mask1_bytes(int p1, int c1) { return (p1 * c1 / 8 + 3) / 4 * 4; }

// byte offsets into the workspace
struct Workspace {
    size_t a1, a2, a3, h;               // bf16 NHWC activations (a3: the last convolution's; two convolutions: no a2)
    size_t a1l, a2l, a3l, hl;           // their low parts (written and read by the forward pass only)
    size_t fcp;                         // fp32 [ksplit][B][512] partial sums of the fc forward GEMM
    size_t zp, cnt;                     // fc_small_kernel: contributions to the head outputs [HID/16][padded B][32], counters
    size_t z;                           // categorical head: fp32 atom logits, rows padded to NHP floats
    size_t ztgt, m;                     // C51: target-net atom logits, projected target
    size_t qt, astar;                   // DQN: target-net Q(s',.) fp32 [B][A]; Double-DQN: online greedy action on s' int32 [B]
    size_t m1, m2, m3;                  // ReLU sign bits of act1, act2 and the last convolution's activations (bit e&7 of byte e>>3, NHWC element e), written by the forward
    size_t dz, dph, dp3, dp2;           // bf16 gradients at pre-activations (d(pre1) never leaves the chip); dp3: the last convolution's
    size_t lossp;                       // fp32 [blocks][4] partial loss sums
    size_t hbp;                         // fp32 [blocks][32 or NHP] partial sums of the head's bias gradient
    size_t pw1, pw2, pw3, pwfc, pwh;    // fp32 weight-gradient partials [split][N*K' + N]
    size_t total;
};
inline int loss_blocks(const Dims &d, int B) {
    const int per = d.small ? loss_block(B) : C51_WAVES * c51_loss_spw(B);
    return (B + per - 1) / per;
}
// `bound`: sizes for which every smaller batch's workspace has room too.
inline Workspace make_workspace(const Dims &d, int B, int mode, bool bound = false) {
    Workspace w{};
    size_t p = 0;
    auto take = [&](size_t bytes) { size_t at = p; p = align_up(p + bytes, 256); return at; };
    const size_t b = (size_t)B, feat = (size_t)d.feat, hid = (size_t)d.hid;
    const bool train = mode == ARN_MODE_TRAIN;
    const size_t e1 = train ? b * d.p1 * d.c1 : 0;                // elements of act1 and act2, which inference keeps on chip
    const size_t e2 = train && d.c3 ? b * d.p2 * d.c2 : 0;
    w.a1 = take(e1 * 2);
    w.a2 = take(e2 * 2);
    // fragment order: whole sample tiles
    const size_t b3 = B <= FC_SMALL_MAX ? align_up(b, fc_small_tile(d.hid, B).rows) : b;
    w.a3 = take(b3 * feat * 2);
    w.h = take(train || !d.small ? b * hid * 2 : 0);
    w.a1l = take(d.c3 ? e1 * 2 : 0);                             // two convolutions: act1 goes to conv2 through LDS
    w.a2l = take(e2 * 2);
    w.a3l = take(train ? b3 * feat * 2 : 0);
    w.hl = take(train || !d.small ? b * hid * 2 : 0);
    // the fused policy/value head kernel always reads fp32 partials; the categorical path only when k is split
    const int ks = std::max(train ? fc_ksplit(d.feat, d.hid, B, false) : 0, fc_ksplit(d.feat, d.hid, B, true));
    const size_t fcp = (size_t)(ks > 1 || d.small ? ks : 0) * b * hid;   // at most 16 ranges, 256 workgroups of 128 x 128 if several
    w.fcp = take((bound ? std::max(std::min(16 * b * hid, (size_t)256 * 128 * 128), d.small ? b * hid : 0) : fcp) * 4);
    if ((bound || fc_small(d.feat, B, true)) && d.small) {
        w.zp = take(hid / 16 * align_up(std::min(b, (size_t)FC_SMALL_MAX), 32) * 32 * 4);
        w.cnt = take((size_t)FC_SMALL_MAX / 16 * 4);
    }
    // categorical head: atom logits of arn_policy_act (arn_policy_forward writes them to its `logits` argument)
    if (mode == ARN_MODE_FORWARD) w.z = take(d.small ? 0 : b * (size_t)d.NHP * 4);
    if (mode == ARN_MODE_TRAIN) {
        w.z = take(d.small ? 0 : b * (size_t)d.NHP * 4);
        if (d.qhead) {
            w.qt = take(b * (size_t)d.A * 4);
            w.astar = take(b * 4);
        }
        if (d.head == ARN_HEAD_C51) {
            w.ztgt = take(b * (size_t)d.NHP * 4);
            w.m = take(b * (size_t)d.atoms * 4);
        }
        w.m1 = take(b * mask1_bytes(d.p1, d.c1));
        w.m2 = take(e2 / 8);
        w.m3 = take(b * feat / 8);
        w.dz = take(b * (size_t)d.NHP * 2);
        w.dph = take(b * hid * 2);
        w.dp3 = take(b * feat * 2);
        w.dp2 = take(e2 * 2);
        size_t lb = (size_t)loss_blocks(d, B);
        Splits s = make_splits(d, B);
        if (bound) {
            for (int end : {512, 2048, 4095}) lb = std::max(lb, (size_t)loss_blocks(d, std::min(B, end)));   // fewer, longer blocks beyond
            s.c1 = std::min(B, CONV_BWD_MOST1);
            s.c2 = std::min(B, CONV_BWD_MOST2);
            s.c3 = d.c3 ? std::min(B, CONV_BWD_MOST2) : 0;
        }
        w.lossp = take(lb * 4 * 4);
        w.hbp = take(lb * (d.small ? 32 : d.NHP) * 4);
        w.pw1 = take((size_t)s.c1 * ((size_t)d.c1 * KW1 + d.c1) * 4);
        w.pw2 = take((size_t)s.c2 * ((size_t)d.c2 * d.kw2 + d.c2) * 4);
        w.pw3 = take((size_t)s.c3 * ((size_t)C3 * KW3 + C3) * 4);
        w.pwfc = take((size_t)s.fc * (hid * feat + hid) * 4);
        w.pwh = take((size_t)s.hd * ((size_t)d.NHP * hid + d.NHP) * 4);
    }
    w.total = p;
    return w;
}

// Sizes reported to callers.  A workspace made for B samples serves every smaller batch too, so what is reported does not
// decrease with B, although what a call needs does now and then (fewer ranges of the fc contraction, fewer partials).
// Calls ask for what they need (make_workspace).
// Inference reports the size that holds every layer's activations: it decides what arn_policy_forward_static accepts.
// The 2-convolution network reports at least the sizes of its embedding in the 104x80 three-convolution network (plus that
// network's flat vector), which are part of the documented interface.
inline Dims embedding_dims(Dims d) {
    d.geom = ARN_GEOM_PAPER;
    set_geometry<GeoPaper>(d);
    return d;
}
inline size_t reported_packed_bytes(const Dims &d) {
    if (d.geom != ARN_GEOM_A3C) return packed_offsets(d).total;
    const Dims e = embedding_dims(d);
    return std::max(packed_offsets(d).total, packed_offsets(e).total + align_up(param_offsets(e).total * 4, 256));
}
// act1 .. h as (hi, lo) pairs, the fc layer's partial sums in up to 16 ranges, the categorical head's logits
inline size_t all_activations_bytes(const Dims &d, int B) {
    size_t p = 0;
    const size_t b = (size_t)B;
    for (size_t n : {b * d.p1 * d.c1, b * d.p2 * d.c2, b * d.feat, b * d.hid}) p += 2 * align_up(n * 2, 256);
    p += align_up(std::max(std::min(16 * b, (size_t)8192), d.small ? b : 0) * d.hid * 4, 256);
    return p + align_up(d.small ? 0 : b * d.NHP * 4, 256);
}
inline size_t reported_workspace_bytes(const Dims &d, int B, int mode) {
    auto bytes = [&](const Dims &x) {
        const size_t need = make_workspace(x, B, mode, true).total;
        return mode == ARN_MODE_TRAIN ? need : std::max(need, all_activations_bytes(x, B));
    };
    if (d.geom != ARN_GEOM_A3C) return bytes(d);
    const Dims e = embedding_dims(d);
    return std::max(bytes(d), bytes(e) + (mode == ARN_MODE_TRAIN ? align_up(param_offsets(e).total * 4, 256) : 0));
}

}  // namespace arn
