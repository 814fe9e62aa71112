// C ABI of the library (declared in include/arn.h): argument checks on the host,
// then a fixed sequence of kernel launches on the caller's stream.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "arn_gemm.h"
#include "arn_layout.h"
#include "arn_problems.h"
#include "arn_pv_head.h"
#include "arn_resident.h"
#include "arn_resident_conv.h"
#include "arn_conv_bwd.h"
#include "arn_dense_bwd.h"
#include "arn_conv23_fwd.h"
#include "arn_infer_fwd.h"
#include "arn_infer_small.h"
#include "arn_conv12_fwd.h"
#include "arn_small_kernels.h"
#include "arn_update.h"

using namespace arn;

// Scratch memory of arn_policy_forward_static, the entry point for callers that cannot allocate: one copy per
// GPU the library runs on, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress (static_scratch_ptr below); kernels receive the device address that call returns.
static __device__ __align__(256) unsigned char scratch[ARN_STATIC_SCRATCH_BYTES];

namespace {

std::mutex g_lazy_mutex;   // guards the lazily filled per-device tables below (first calls from several host threads)

inline bool aligned(const void *p, size_t a) { return p && (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline bool known_head(int k) { return k == ARN_HEAD_PV || k == ARN_HEAD_C51 || k == ARN_HEAD_Q || k == ARN_HEAD_DUEL; }

// gfx950 check, cached per device
int check_arch() {
    static int cached[64];   // 0 unknown, 1 ok, -1 wrong arch, -2 hip error
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return ARN_EHIP;
    if (dev < 0 || dev >= 64) return ARN_EHIP;
    std::lock_guard<std::mutex> lock(g_lazy_mutex);
    if (cached[dev] == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) cached[dev] = -2;
        else cached[dev] = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : -1;
    }
    return cached[dev] == 1 ? ARN_OK : (cached[dev] == -1 ? ARN_EARCH : ARN_EHIP);
}

inline int launched() { return hipGetLastError() == hipSuccess ? ARN_OK : ARN_EHIP; }

// Optional instrumentation (arn_profile_enable): a pair of HIP events around every launch.
struct ProfRecord {
    const char *name;
    hipEvent_t start, stop;
};
bool g_prof_on = false;
std::vector<ProfRecord> g_prof;
struct ProfScope {
    hipStream_t s;
    bool on;
    ProfScope(const char *name, hipStream_t stream) : s(stream), on(g_prof_on) {
        if (!on) return;
        ProfRecord r{name, nullptr, nullptr};
        if (hipEventCreate(&r.start) != hipSuccess || hipEventCreate(&r.stop) != hipSuccess) { on = false; return; }
        (void)hipEventRecord(r.start, s);
        g_prof.push_back(r);
    }
    ~ProfScope() {
        if (on) (void)hipEventRecord(g_prof.back().stop, s);
    }
};

inline unsigned cdiv(long a, long b) { return (unsigned)((a + b - 1) / b); }

// Device address of this GPU's copy of `scratch`, looked up once per device with that device current.
void *static_scratch_ptr() {
    static void *per_dev[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(g_lazy_mutex);
    if (!per_dev[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        per_dev[dev] = ptr;
    }
    return per_dev[dev];
}

template <bool SPLIT, class P>
void launch_nt(const char *name, const P &p, int N, int z, hipStream_t s) {
    ProfScope ps(name, s);
    hipLaunchKernelGGL((gemm_nt_kernel<P, SPLIT>), dim3(cdiv(p.M, P::BM), cdiv(N, NT_BN), z), dim3(NT_THREADS), 0, s, p);
}

// rows of the batch per split of a weight-gradient contraction: whole k-tiles
inline int rows_per_split(long M, int splits) { return (int)((M + splits - 1) / splits + 63) / 64 * 64; }

// sample-resident convolution: a fixed, contiguous range of samples per workgroup
struct ResidentGrid {
    int spw, wgs, parts;   // samples per workgroup, sample ranges, workgroups that share a range
};
template <class C>
ResidentGrid resident_grid(int B) {
    const int groups = (B + C::G - 1) / C::G;
    const int target = C::NBUF == 1 && ResWaves<C>::value == 4 ? 512 : 256;   // single-buffered four-wavefront kernels share a CU
    ResidentGrid g;
    g.spw = resident_spw(groups, target) * C::G;
    // with few sample groups, the position tiles of a group are dealt to several workgroups
    constexpr int tiles = (C::G * C::P + 15) / 16;
    g.wgs = (int)cdiv(B, g.spw);
    g.parts = 128 / g.wgs;   // every extra workgroup repeats the weight fetch and the staging: measured to pay only up to about 128 workgroups
    g.parts = g.parts < 1 ? 1 : g.parts > tiles ? tiles : g.parts;
    return g;
}
template <class C>
void launch_resident(const char *name, const typename C::Args &a, int B, hipStream_t s) {
    ProfScope ps(name, s);
    const ResidentGrid g = resident_grid<C>(B);
    hipLaunchKernelGGL(resident_conv_kernel<C>, dim3(g.wgs, g.parts), dim3(64 * ResWaves<C>::value), 0, s, a, B, g.spw);
}

struct Packed {   // typed views of the packed blob
    const __bf16 *w1, *w2, *w3, *wfc, *wh, *whd, *wfcd, *w3d, *w2d;
    const __bf16 *w1l, *w2l, *w3l, *wfcl, *whl;
    const _Float16 *w1h, *w2h, *w3h, *wfch;   // fp16 forward layouts
    const float *b1, *b2, *b3, *bfc, *bh;
};
Packed view_packed(const void *blob, const Dims &d) {
    const PackedOffsets o = packed_offsets(d);
    const char *b = (const char *)blob;
    Packed p;
    p.w1 = (const __bf16 *)(b + o.w1);
    p.w2 = (const __bf16 *)(b + o.w2);
    p.w3 = (const __bf16 *)(b + o.w3);
    p.wfc = (const __bf16 *)(b + o.wfc);
    p.wh = (const __bf16 *)(b + o.wh);
    p.b1 = (const float *)(b + o.b1);
    p.b2 = (const float *)(b + o.b2);
    p.b3 = (const float *)(b + o.b3);
    p.bfc = (const float *)(b + o.bfc);
    p.bh = (const float *)(b + o.bh);
    p.whd = (const __bf16 *)(b + o.whd);
    p.wfcd = (const __bf16 *)(b + o.wfcd);
    p.w3d = (const __bf16 *)(b + o.w3d);
    p.w2d = (const __bf16 *)(b + o.w2d);
    p.w1l = (const __bf16 *)(b + o.w1l);
    p.w2l = (const __bf16 *)(b + o.w2l);
    p.w3l = (const __bf16 *)(b + o.w3l);
    p.wfcl = (const __bf16 *)(b + o.wfcl);
    p.whl = (const __bf16 *)(b + o.whl);
    p.w1h = (const _Float16 *)(b + o.w1h);
    p.w2h = (const _Float16 *)(b + o.w2h);
    p.w3h = (const _Float16 *)(b + o.w3h);
    p.wfch = (const _Float16 *)(b + o.wfch);
    return p;
}

// Arguments of the head kernels that the entry points share.  ks: k ranges of the fc partial sums.
PvHeadArgs pv_head_args(const Dims &d, const Packed &w, int B, char *ws, const Workspace &o, int ks) {
    PvHeadArgs p = {};
    p.partial = (const float *)(ws + o.fcp); p.ks = ks; p.bfc = w.bfc;
    p.wh = w.wh; p.whl = w.whl; p.bh = w.bh; p.B = B; p.A = d.A;
    p.qmode = d.head == ARN_HEAD_Q ? 1 : d.head == ARN_HEAD_DUEL ? 2 : 0;
    return p;
}
// Samples per workgroup of the head kernel in the inference calls: small batches are spread over more CUs
inline int infer_rows_per_block(int B) { return B <= 512 ? 4 : B <= 4096 ? 8 : PVH_ROWS; }

// Calls f with the geometry of d.
template <class F>
void with_geometry(const Dims &d, F f) {
    if (d.geom == ARN_GEOM_PAPER) f(GeoPaper());
    else if (d.geom == ARN_GEOM_A3C) f(GeoA3c());
    else f(Geo84());
}

// Calls f with the positions per workgroup tile of a dense contraction over M rows and N columns (dense_tile).
template <class F>
void with_tile(long M, int N, F f) {
    const int tile = dense_tile(M, N);
    if (tile == 128) f(std::integral_constant<int, 128>());
    else if (tile == 64) f(std::integral_constant<int, 64>());
    else f(std::integral_constant<int, 32>());
}

template <class G, bool F16, int MODE>
void launch_fc_small(const char *name, const FcSmallArgs &p, int B, hipStream_t s) {
    ProfScope ps(name, s);
    auto launch = [&](auto nt, auto mt) {
        constexpr int NT = decltype(nt)::value, MT = decltype(mt)::value;
        hipLaunchKernelGGL((fc_small_kernel<G::FEAT, G::NHID, NT, MT, F16, MODE>), dim3(G::NHID / (16 * NT), cdiv(B, 16 * MT)),
                           dim3(fc_small_threads<G::FEAT>()), 0, s, p);
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;
    const FcTile t = fc_small_tile(G::NHID, B);
    if (t.rows == 16) launch(One(), One());
    else if (t.units == 16) launch(One(), Two());
    else launch(Two(), Two());
}

// fc layer and, for the categorical head, the head GEMM.  F16: act3 and the fc weights are fp16 and the layer is one
// product (no-gradient forward); otherwise three bf16 products.  `head`: no-gradient forward with one of the small
// heads: its outputs are written too.  Without it (gradient step) the caller launches pv_head_kernel on the fc sums.
template <class G, bool F16>
void fc_and_head_launches(const Dims &d, const Packed &w, int B, char *ws, const Workspace &o, float *z_out,
                          int zstride, PvHeadArgs *head, hipStream_t s) {
    __bf16 *a3 = (__bf16 *)(ws + o.a3), *a3l = (__bf16 *)(ws + o.a3l);
    __bf16 *h = (__bf16 *)(ws + o.h), *hl = (__bf16 *)(ws + o.hl);
    if (fc_small(G::FEAT, B, F16)) {
        FcSmallArgs p = {};
        p.act = a3; p.act_lo = a3l; p.w = F16 ? (const void *)w.wfch : (const void *)w.wfc; p.w_lo = w.wfcl; p.B = B;
        p.partial = (float *)(ws + o.fcp); p.bias = w.bfc; p.h = h; p.h_lo = hl;
        if (!d.small) {
            launch_fc_small<G, F16, FC_HIDDEN>("fc_fwd", p, B, s);
        } else if constexpr (F16) {
            p.head = *head; p.zp = (float *)(ws + o.zp); p.counters = (unsigned *)(ws + o.cnt);
            launch_fc_small<G, F16, FC_HEAD>("fc_head", p, B, s);
        } else {
            launch_fc_small<G, F16, FC_PARTIAL>("fc_fwd", p, B, s);
        }
    } else {
        const int ksplit = fc_ksplit(G::FEAT, G::NHID, B, F16);
        const bool partial = ksplit > 1 || d.small;
        auto launch = [&](auto bm, auto to_partial) {
            constexpr int BM = decltype(bm)::value;
            constexpr bool P = decltype(to_partial)::value;
            typename std::conditional<F16, FcFwdF16T<G::FEAT, G::NHID, BM, P>, FcFwdT<G::FEAT, G::NHID, BM, P>>::type p;
            p.in = a3; p.in_lo = a3l; p.M = B; p.w = F16 ? (const __bf16 *)w.wfch : w.wfc; p.w_lo = w.wfcl; p.bias = w.bfc;
            p.out = h; p.out_lo = hl; p.ksplit = ksplit; p.partial = (float *)(ws + o.fcp);
            launch_nt<!F16>("fc_fwd", p, G::NHID, ksplit, s);
        };
        // a tile of 64 is one of at most 64 tiles: its contraction is always cut
        if (fc_tile(G::NHID, B) != 128) launch(Count<64>(), std::true_type());
        else if (partial) launch(Count<128>(), std::true_type());
        else launch(Count<128>(), std::false_type());
        if (ksplit > 1 && !d.small) {
            ProfScope ps("fc_finish", s);
            const long total = (long)B * G::NHID;
            hipLaunchKernelGGL(fc_finish_kernel, dim3(cdiv(total / 4, 256)), dim3(256), 0, s, (const float *)(ws + o.fcp), ksplit,
                               w.bfc, h, hl, G::NHID, total);
        }
        if (d.small && head) {
            ProfScope ps("pv_head", s);
            head->ks = ksplit;
            head->rpb = infer_rows_per_block(B);
            hipLaunchKernelGGL((pv_head_kernel<false, G::NHID>), dim3(cdiv(B, head->rpb)), dim3(PVH_THREADS), 0, s, *head);
        }
    }
    if (d.head == ARN_HEAD_C51) {
        auto launch = [&](auto bm) {
            HeadFwdC51<G::NHID, decltype(bm)::value> p;
            p.in = h; p.in_lo = hl; p.M = B; p.w = w.wh; p.w_lo = w.whl; p.bias = w.bh; p.z = z_out; p.NHP = d.NHP; p.ZW = d.NH;
            p.ZS = zstride;
            launch_nt<true>("head_fwd", p, d.NHP, 1, s);
        };
        with_tile(B, d.NHP, launch);
    }
}

// Which configurations of the sample-resident kernels a geometry uses: the 84x84 network has hand-laid LDS
// images, any other geometry the ones whose padding is computed from its map sizes.
template <class G>
struct ConvConfigs {
    typedef ResConv2FwdGeo<G> Fwd2;
    typedef ResConv3FwdGeo<G> Fwd3;
    typedef ResConv3DgradGeo<G> Dgrad3;
    typedef ResConv2DgradGeo<G> Dgrad2;
    static int conv1_parts(int) { return 1; }
    // the three convolutions one after the other in one launch (conv123_chain_kernel), from 65 samples on: below, several
    // workgroups share a sample of conv2 and conv3
    static constexpr bool CHAINS = true;
    static bool chain(int B) { return B >= 65; }
    // conv2 -> conv3 through LDS needs both layers' images in one CU's LDS: not with the bordered images of this geometry
    static bool fused_conv23(int) { return false; }
    static void launch_conv23(const Conv23Args &, int, int, hipStream_t) {}
    static void launch_conv123(const uint8_t *, const __bf16 *, const __bf16 *, const float *, uint8_t *, const Conv23Args &, int,
                               int, hipStream_t) {}
};
template <>
struct ConvConfigs<GeoA3c> {
    typedef ResConv2FwdGeo<GeoA3c> Fwd2;
    typedef NoConv3 Fwd3;
    typedef ResConv2DgradGeo<GeoA3c> Dgrad2;
};
template <>
struct ConvConfigs<Geo84> {
    typedef ResConv2Fwd Fwd2;
    typedef ResConv3Fwd Fwd3;
    typedef ResConv3Dgrad Dgrad3;
    typedef ResConv2Dgrad Dgrad2;
    static constexpr bool CHAINS = false;
    // few samples: three workgroups share one (one workgroup fits per CU)
    static int conv1_parts(int B) { return 3 * B <= 256 ? 3 : 1; }
    // one workgroup per sample range and no tile splitting: measured equal to the two kernels at B = 64, faster above
    static bool fused_conv23(int B) { return B >= 64; }
    static void launch_conv23(const Conv23Args &p, int B, int spw, hipStream_t s) {
        hipLaunchKernelGGL((conv23_fwd_fused_kernel<ResConv2Fwd, ResConv3Fwd>), dim3((B + spw - 1) / spw), dim3(C23_THREADS), 0,
                           s, p, B, spw);
    }
    static void launch_conv123(const uint8_t *obs, const __bf16 *w1, const __bf16 *w1l, const float *b1, uint8_t *m1,
                               const Conv23Args &p, int B, int spw, hipStream_t s) {
        hipLaunchKernelGGL((conv123_fwd_kernel<Geo84, ResConv2Fwd, ResConv3Fwd>), dim3((B + spw - 1) / spw), dim3(C23_THREADS),
                           0, s, obs, w1, w1l, b1, m1, p, B, spw);
    }
};

// Forward pass of a gradient step for geometry G in three-product bf16 precision (conv1's pixel operand is exact: two
// products), with the ReLU sign bits of every convolution for the backward pass.  C51: z_out = atom logits, rows of zstride
// floats.  PV, Q, DUEL: stops after the fc GEMM, whose fp32 sums (o.fcp) the fused head kernel consumes.
template <class G>
void forward_trunk(const Dims &d, const Packed &w, const uint8_t *obs, int B, char *ws, const Workspace &o,
                   float *z_out, int zstride, hipStream_t s) {
    typedef ConvConfigs<G> Cfg;
    __bf16 *a1 = (__bf16 *)(ws + o.a1), *a2 = (__bf16 *)(ws + o.a2), *a3 = (__bf16 *)(ws + o.a3);
    __bf16 *a1l = (__bf16 *)(ws + o.a1l), *a2l = (__bf16 *)(ws + o.a2l), *a3l = (__bf16 *)(ws + o.a3l);
    uint8_t *m1 = (uint8_t *)(ws + o.m1), *m2 = (uint8_t *)(ws + o.m2), *m3 = (uint8_t *)(ws + o.m3);
    if constexpr (!G::HAS3) {
        ProfScope ps("conv12_fwd", s);
        Conv12Args p;
        p.obs = obs; p.w1 = w.w1; p.w1_lo = w.w1l; p.w2 = w.w2; p.w2_lo = w.w2l; p.b1 = w.b1; p.b2 = w.b2;
        p.a1 = a1; p.m1 = m1; p.a2 = a3; p.a2_lo = a3l; p.m2 = m3; p.frag = fc_small(G::FEAT, B, false);
        const BandPlan bp = band_plan<G>(B);
        const int spw = resident_spw(B, 256);
        hipLaunchKernelGGL((conv12_fwd_kernel<G, typename Cfg::Fwd2>), dim3(cdiv(B, spw) * bp.bands), dim3(C12_THREADS), 0, s, p, B,
                           spw, bp.rows, bp.bands);
    } else {
        typename Cfg::Fwd2::Args p2;
        p2.in = a1; p2.in_lo = a1l; p2.w = w.w2; p2.w_lo = w.w2l; p2.mask = nullptr; p2.bias = w.b2; p2.out = a2; p2.out_lo = a2l;
        p2.mask_out = m2;
        typename Cfg::Fwd3::Args p3;
        p3.in = a2; p3.in_lo = a2l; p3.w = w.w3; p3.w_lo = w.w3l; p3.mask = nullptr; p3.bias = w.b3; p3.out = a3; p3.out_lo = a3l;
        p3.mask_out = m3; p3.frag = fc_small(G::FEAT, B, false);
        const int spw = resident_spw(B, 256);
        auto chain_launch = [&]() {     // whether it launched them
            if constexpr (Cfg::CHAINS) {
                if (Cfg::chain(B)) {
                    ProfScope ps("conv123_fwd", s);
                    hipLaunchKernelGGL((conv123_chain_kernel<G, typename Cfg::Fwd2, EightWaves<typename Cfg::Fwd3>>), dim3(cdiv(B, spw)),
                                       dim3(RES_THREADS), 0, s, obs, w.w1, w.w1l, w.b1, m1, p2, p3, B, spw);
                    return true;
                }
            }
            return false;
        };
        if (!chain_launch()) {
            const bool chained = Cfg::fused_conv23(B) && Cfg::conv1_parts(B) == 1;
            if (!chained) {
                ProfScope ps("conv1_fwd", s);
                hipLaunchKernelGGL(conv1_fwd_resident_kernel<G>, dim3(cdiv(B, spw), Cfg::conv1_parts(B)), dim3(RES_THREADS), 0, s,
                                   obs, w.w1, w.w1l, w.b1, a1, a1l, m1, B, spw);
            }
            if (Cfg::fused_conv23(B)) {
                // conv2 and conv3 in one kernel: act2 passes through LDS; with one workgroup per sample range in conv1 too,
                // conv1 runs in the same launch, ahead of them in every workgroup
                ProfScope ps(chained ? "conv123_fwd" : "conv23_fwd", s);
                Conv23Args p;
                p.a1 = a1; p.a1_lo = a1l; p.w2 = w.w2; p.w2_lo = w.w2l; p.w3 = w.w3; p.w3_lo = w.w3l; p.b2 = w.b2; p.b3 = w.b3;
                p.a2 = a2; p.a3 = a3; p.a3_lo = a3l;
                p.m2 = m2; p.m3 = m3;
                p.frag = fc_small(G::FEAT, B, false);
                if (chained) Cfg::launch_conv123(obs, w.w1, w.w1l, w.b1, m1, p, B, spw, s);
                else Cfg::launch_conv23(p, B, spw, s);
            } else {
                launch_resident<typename Cfg::Fwd2>("conv2_fwd", p2, B, s);
                launch_resident<typename Cfg::Fwd3>("conv3_fwd", p3, B, s);
            }
        }
    }
    fc_and_head_launches<G, false>(d, w, B, ws, o, z_out, zstride, nullptr, s);
}

// one workgroup per range of samples; the software-pipelined variant where its 17 KB of weights and biases fit beside the
// LDS images (84x84)
template <class G, bool FRAG>
void launch_infer_conv(const InferConvArgs &p, int B, hipStream_t s) {
    typedef typename ConvConfigs<G>::Fwd2 F2;
    typedef typename ConvConfigs<G>::Fwd3 F3;
    const int spw = resident_spw(B, 256);
    if constexpr (infer_pipelined_fits<G, F2, F3>())
        hipLaunchKernelGGL((infer_conv_pipelined_kernel<G, F2, F3, FRAG>), dim3(cdiv(B, spw)), dim3(INF_THREADS), 0, s, p, B, spw);
    else
        hipLaunchKernelGGL((infer_conv_kernel<G, F2, F3, FRAG>), dim3(cdiv(B, spw)), dim3(INF_THREADS), 0, s, p, B, spw);
}

// Forward pass that carries no gradient (action selection): the convolutions in one kernel and one fp16 product per
// layer, act3 in fp16, then the fc layer in fp16.  C51: z_out = atom logits, rows of zstride floats; the other heads
// write what `head` asks for.
template <class G>
void infer_trunk(const Dims &d, const Packed &w, const uint8_t *obs, int B, char *ws, const Workspace &o,
                 float *z_out, int zstride, PvHeadArgs *head, hipStream_t s) {
    typedef ConvConfigs<G> Cfg;
    {
        ProfScope ps("conv_infer", s);
        InferConvArgs p;
        p.obs = obs; p.w1 = w.w1h; p.w2 = w.w2h; p.w3 = w.w3h; p.b1 = w.b1; p.b2 = w.b2; p.b3 = w.b3;
        p.a3 = (_Float16 *)(ws + o.a3);
        p.counters = (unsigned *)(ws + o.cnt);
        p.n_counters = fc_small(G::FEAT, B, true) && d.small ? (int)cdiv(B, fc_small_tile(G::NHID, B).rows) : 0;
        const BandPlan bp = band_plan<G>(B);
        if (bp.bands > 1)   // at most 128 samples
            hipLaunchKernelGGL((infer_conv_band_kernel<G, typename Cfg::Fwd2, typename Cfg::Fwd3>), dim3(B * bp.bands),
                               dim3(INF_THREADS), 0, s, p, bp.rows, bp.bands);
        else if (fc_small(G::FEAT, B, true)) launch_infer_conv<G, true>(p, B, s);
        else launch_infer_conv<G, false>(p, B, s);
    }
    fc_and_head_launches<G, true>(d, w, B, ws, o, z_out, zstride, head, s);
}
void infer_launches(const Dims &d, const Packed &w, const uint8_t *obs, int B, char *ws, const Workspace &o,
                    float *z_out, int zstride, PvHeadArgs *head, hipStream_t s) {
    with_geometry(d, [&](auto g) { infer_trunk<decltype(g)>(d, w, obs, B, ws, o, z_out, zstride, head, s); });
}
void forward_launches(const Dims &d, const Packed &w, const uint8_t *obs, int B, char *ws, const Workspace &o,
                      float *z_out, int zstride, hipStream_t s) {
    with_geometry(d, [&](auto g) { forward_trunk<decltype(g)>(d, w, obs, B, ws, o, z_out, zstride, s); });
}

// Backward pass below d(pre_fc) for geometry G, in four launches: the dense layers' gradients, conv3's input gradient,
// the convolutions' weight gradients (with conv2's input gradient), the sums of all weight-gradient partials.
// Within a launch, pieces of work that do not depend on each other are ranges of workgroups.  A launch costs about 4 us
// on the GPU and 3 us on the host however small it is, a cross-stream event about 6 us on both streams: with the dense
// weight gradients and five short kernels on a second stream the step took 139 us at 333 samples (host 105 us), this
// way 126 (host 40); from 2048 samples up the two are level.
template <class G>
void backward_trunk(const Dims &d, const Packed &w, const uint8_t *obs, int B, char *ws, const Workspace &o, const LossTotals &loss,
                    int loss_blocks, float *dW, hipStream_t s) {
    typedef ConvConfigs<G> Cfg;
    const ParamOffsets po = param_offsets(d);
    const Splits sp = make_splits(d, B);
    __bf16 *h = (__bf16 *)(ws + o.h), *dz = (__bf16 *)(ws + o.dz);
    float *parth = (float *)(ws + o.pwh);
    __bf16 *a1 = (__bf16 *)(ws + o.a1), *a2 = (__bf16 *)(ws + o.a2), *a3 = (__bf16 *)(ws + o.a3);
    __bf16 *dph = (__bf16 *)(ws + o.dph), *dp3 = (__bf16 *)(ws + o.dp3);
    __bf16 *dp2 = (__bf16 *)(ws + o.dp2);
    float *part1 = (float *)(ws + o.pw1), *part2 = (float *)(ws + o.pw2), *part3 = (float *)(ws + o.pw3);
    float *partfc = (float *)(ws + o.pwfc);
    {
        auto launch = [&](auto bm, auto units) {
            typedef FcDgradT<G::FEAT, G::NHID, decltype(bm)::value> Dg;
            Dg dg;
            typedef FcWgrad<G::FEAT, G::NHID, decltype(units)::value> FcW;
            typedef HeadWgrad<G::NHID> HeadW;
            dg.in = dph; dg.M = B; dg.w = w.wfcd; dg.maskbits = (const uint8_t *)(ws + o.m3); dg.out = dp3;
            DenseBackwardArgs<Dg, FcW, HeadW> p;
            p.dg = dg;
            p.dg_x = cdiv(B, Dg::BM); p.dg_blocks = p.dg_x * cdiv(G::FEAT, NT_BN);
            p.wg.in = a3; p.wg.M = B; p.wg.frag = fc_small(G::FEAT, B, false); p.wg.dy = dph;
            p.wg_part = partfc; p.wg_rows = rows_per_split(B, sp.fc);
            p.wg_blocks = (G::FEAT / FcW::BK2) * (G::NHID / FcW::BN1) * sp.fc;
            p.hw.in = h; p.hw.M = B; p.hw.N1 = d.NHP; p.hw.dy = dz;
            p.hw_part = parth; p.hw_rows = rows_per_split(B, sp.hd);
            p.hw_blocks = (G::NHID / HeadW::BK2) * (d.NHP / HeadW::BN1) * sp.hd;
            p.loss = loss;
            ProfScope ps("dense_bwd", s);
            hipLaunchKernelGGL((dense_backward_kernel<Dg, FcW, HeadW>), dim3(p.dg_blocks + p.wg_blocks + p.hw_blocks + 1),
                               dim3(DENSE_THREADS), 0, s, p);
        };
        with_tile(B, G::FEAT, [&](auto bm) {
            if constexpr (decltype(bm)::value == 128 && G::NHID > 256) {
                if (fc_wgrad_units(G::FEAT, G::NHID, B) == 256) return launch(bm, Count<256>());
            }
            launch(bm, Count<128>());
        });
    }
    if constexpr (G::HAS3) {
        typename Cfg::Dgrad3::Args p;
        p.in = dp3; p.in_lo = nullptr; p.w = w.w3d; p.w_lo = nullptr; p.mask = (const uint8_t *)(ws + o.m2); p.out = dp2;
        launch_resident<typename Cfg::Dgrad3>("conv3_dgrad", p, B, s);
    }
    {
        // One launch for everything that is left once d(pre2) exists: conv2's input gradient fused with conv1's
        // weight gradient (conv1's input is data, so d(pre1) has this one consumer and stays in LDS), and the
        // weight gradients of conv2 and conv3 -- three ranges of workgroups, longest first.
        ProfScope ps("conv_bwd", s);
        ConvBackwardArgs p;
        p.obs = obs; p.dp2 = G::HAS3 ? dp2 : dp3; p.w2d = w.w2d; p.mask1 = (const uint8_t *)(ws + o.m1); p.part1 = part1;
        p.a1 = a1; p.a2 = a2; p.dp3 = dp3; p.part2 = part2; p.part3 = part3;
        p.B = B; p.n1 = sp.c1; p.n2 = sp.c2;
        const ConvBwdSplit cs = conv_bwd_split(d, B);
        p.spw1 = cs.spw1; p.spw2 = cs.spw2; p.spw3 = cs.spw3;
        hipLaunchKernelGGL((conv_backward_kernel<G, typename Cfg::Dgrad2>), dim3(sp.c1 + sp.c2 + sp.c3),
                           dim3(ConvBackward<G, typename Cfg::Dgrad2>::THREADS), 0, s, p);
    }
    {
        // one launch adds the partials of every layer (x = u8/255: conv1's pixel scale comes out of the contraction and
        // is applied here; bias gradients have no such factor)
        ReduceAllPlan<G> pl;
        pl.conv1 = make_reduce(UnmapConv1<G::NC1>{(long)po.w1, (long)po.b1}, part1, (long)G::NC1 * KW1, G::NC1, sp.c1, 1.f / 255.f);
        pl.conv2 = make_reduce(UnmapConv<G::NC1, K2, G::NC2>{(long)po.w2, (long)po.b2}, part2, (long)G::NC2 * G::KW2, G::NC2, sp.c2);
        pl.conv3 = make_reduce(UnmapConv<C2, K3, C3>{(long)po.w3, (long)po.b3}, part3, (long)C3 * KW3, C3, sp.c3);
        pl.head = make_reduce(UnmapHead<G::NHID>{head_rows<G::NHID>(d, po), d.NHP}, parth, (long)d.NHP * G::NHID, d.NHP, sp.hd);
        // the head's bias gradient: the loss kernel's fp32 block partials, added in block order
        pl.head_bias = make_reduce(UnmapHeadBias<G::NHID>{head_rows<G::NHID>(d, po)}, (const float *)(ws + o.hbp), 0, d.small ? 32 : d.NHP, loss_blocks);
        pl.n1 = reduce_blocks(pl.conv1); pl.n2 = reduce_blocks(pl.conv2); pl.n3 = G::HAS3 ? reduce_blocks(pl.conv3) : 0;
        pl.nh = reduce_blocks(pl.head);
        pl.fc_part = partfc; pl.fc_w = (long)po.wfc; pl.fc_b = (long)po.bfc; pl.fc_splits = sp.fc;
        ProfScope ps("reduce", s);
        hipLaunchKernelGGL(reduce_all_kernel<G>, dim3(G::NHID + 1 + pl.n1 + pl.n2 + pl.n3 + pl.nh + reduce_blocks(pl.head_bias)), dim3(256), 0, s, pl, dW);
    }
}

// Lays the flat fp32 parameters out in every packed form, one launch.
void launch_pack_all(const Dims &d, const float *w_fp32, void *w_packed, hipStream_t s) {
    ProfScope ps("pack_all", s);
    with_geometry(d, [&](auto g) {
        typedef decltype(g) G;
        const PackPlan<G> pl = make_pack_plan<G>(d, w_packed);
        hipLaunchKernelGGL(pack_all_kernel<G>, dim3(pl.blocks), dim3(256), 0, s, pl, w_fp32);
    });
}

// Shared argument checks of the update entry points.  Returns ARN_OK and fills *d_out when a repack is asked for.
int check_update(size_t n, const arn_config *cfg, const void *w_packed, bool *repack, Dims *d_out) {
    if (n == 0 || n > ((size_t)1 << 40)) return ARN_EINVAL;
    *repack = w_packed != nullptr;
    if (*repack) {
        if (!cfg) return ARN_EINVAL;
        if (!known_head(cfg->head_kind)) return ARN_EKIND;
        *d_out = make_dims(cfg);
        if (!d_out->ok) return ARN_ESHAPE;
        if (n != param_offsets(*d_out).total) return ARN_ESHAPE;
        if (!aligned(w_packed, 256)) return ARN_EINVAL;
    }
    return ARN_OK;
}
inline bool unit_interval(float b) { return b >= 0.f && b < 1.f; }

// One launch: the rule alone, or the rule and every packed copy of the new parameters.
template <int RULE>
void launch_update(const char *name, const UpdateArgs &p, bool repack, const Dims &d, void *w_packed, hipStream_t s) {
    ProfScope ps(name, s);
    if (!repack) {
        hipLaunchKernelGGL(update_kernel<RULE>, dim3((unsigned)((p.n + 1023) / 1024)), dim3(256), 0, s, p);
        return;
    }
    with_geometry(d, [&](auto g) {
        typedef decltype(g) G;
        const PackPlan<G> pl = make_pack_plan<G>(d, w_packed);
        hipLaunchKernelGGL((update_pack_kernel<RULE, G>), dim3(update_pack_blocks(pl)), dim3(256), 0, s, pl, p);
    });
}

}  // namespace

extern "C" {

const char *arn_status_string(int status) {
    switch (status) {
        case ARN_OK: return "ok";
        case ARN_EINVAL: return "invalid argument (null or misaligned pointer, B <= 0 or B > 2^20)";
        case ARN_ESHAPE: return "unsupported shape (num_actions, num_atoms or head for this call)";
        case ARN_EKIND: return "unknown head_kind, loss_kind or mode";
        case ARN_EWORKSPACE: return "workspace too small";
        case ARN_EARCH: return "device is not gfx950";
        case ARN_EHIP: return "HIP runtime error";
        case ARN_ESTATIC: return "batch too large for the library's static scratch buffer (arn_policy_forward_static)";
        default: return "unknown status";
    }
}

size_t arn_param_count(const arn_config *cfg) {
    const Dims d = make_dims(cfg);
    return d.ok ? param_offsets(d).total : 0;
}

size_t arn_packed_bytes(const arn_config *cfg) {
    const Dims d = make_dims(cfg);
    return d.ok ? reported_packed_bytes(d) : 0;
}

size_t arn_workspace_bytes(const arn_config *cfg, int B, int mode) {
    const Dims d = make_dims(cfg);
    if (!d.ok || B <= 0 || B > (1 << 20) || (mode != ARN_MODE_FORWARD && mode != ARN_MODE_TRAIN)) return 0;
    return reported_workspace_bytes(d, B, mode);
}

int arn_weights_prepare(const arn_config *cfg, const float *w_fp32, void *w_packed, void *stream) {
    if (!cfg) return ARN_EINVAL;
    if (!known_head(cfg->head_kind)) return ARN_EKIND;
    const Dims d = make_dims(cfg);
    if (!d.ok) return ARN_ESHAPE;
    if (!aligned(w_fp32, 16) || !aligned(w_packed, 256)) return ARN_EINVAL;
    if (int e = check_arch()) return e;
    hipStream_t s = (hipStream_t)stream;
    launch_pack_all(d, w_fp32, w_packed, s);
    return launched();
}

namespace {
// Argument checks shared by arn_policy_forward and arn_policy_forward_static; fills *d_out.
int check_policy_forward(const arn_config *cfg, const void *w_packed, const uint8_t *obs, int B, float *logits,
                         float *value, float *probs, int32_t *greedy, Dims *d_out) {
    if (!cfg || B <= 0 || B > (1 << 20)) return ARN_EINVAL;
    if (!known_head(cfg->head_kind)) return ARN_EKIND;
    const Dims d = make_dims(cfg);
    if (!d.ok) return ARN_ESHAPE;
    if (!aligned(w_packed, 256) || !aligned(obs, 16) || !aligned(logits, 16)) return ARN_EINVAL;
    if (d.small && !aligned(value, 16)) return ARN_EINVAL;
    if ((value && !aligned(value, 16)) || (probs && !aligned(probs, 16)) || (greedy && !aligned(greedy, 16)))
        return ARN_EINVAL;
    if (d.qhead && probs) return ARN_ESHAPE;
    *d_out = d;
    return ARN_OK;
}

// The launches of one inference call; `ws` holds make_workspace(d, B, ARN_MODE_FORWARD).total bytes.
int policy_forward_launches(const arn_config *cfg, const Dims &d, const Workspace &o, const void *w_packed,
                            const uint8_t *obs, int B, float *logits, float *value, float *probs, int32_t *greedy,
                            char *ws, hipStream_t s) {
    const Packed w = view_packed(w_packed, d);
    PvHeadArgs p = pv_head_args(d, w, B, ws, o, 1);
    p.logits = logits; p.value = value; p.probs = probs; p.greedy = greedy;
    infer_launches(d, w, obs, B, ws, o, logits, d.NH, &p, s);
    if (!d.small && (value || probs || greedy)) {
        ProfScope ps("c51_dist", s);
        hipLaunchKernelGGL(c51_dist_kernel, dim3(cdiv(B, C51_WAVES)), dim3(64 * C51_WAVES), 0, s, logits, d.NH, B, d.A,
                           d.atoms, cfg->v_min, cfg->v_max, cfg->gamma, (const float *)nullptr,
                           (const uint8_t *)nullptr, probs, value, greedy, (float *)nullptr);
    }
    return launched();
}
}  // namespace

int arn_policy_forward(const arn_config *cfg, const void *w_packed, const uint8_t *obs, int B, float *logits,
                       float *value, float *probs, int32_t *greedy, void *workspace, size_t workspace_bytes,
                       void *stream) {
    Dims d;
    if (int e = check_policy_forward(cfg, w_packed, obs, B, logits, value, probs, greedy, &d)) return e;
    if (!aligned(workspace, 256)) return ARN_EINVAL;
    const Workspace o = make_workspace(d, B, ARN_MODE_FORWARD);
    if (workspace_bytes < o.total) return ARN_EWORKSPACE;
    if (int e = check_arch()) return e;
    return policy_forward_launches(cfg, d, o, w_packed, obs, B, logits, value, probs, greedy, (char *)workspace,
                                   (hipStream_t)stream);
}

int arn_policy_forward_static(const arn_config *cfg, const void *w_packed, const uint8_t *obs, int B, float *logits,
                              float *value, float *probs, int32_t *greedy, void *stream) {
    Dims d;
    if (int e = check_policy_forward(cfg, w_packed, obs, B, logits, value, probs, greedy, &d)) return e;
    const Workspace o = make_workspace(d, B, ARN_MODE_FORWARD);
    if (reported_workspace_bytes(d, B, ARN_MODE_FORWARD) > (size_t)ARN_STATIC_SCRATCH_BYTES) return ARN_ESTATIC;
    if (int e = check_arch()) return e;
    void *ptr = static_scratch_ptr();
    if (!ptr) return ARN_EHIP;
    return policy_forward_launches(cfg, d, o, w_packed, obs, B, logits, value, probs, greedy, (char *)ptr,
                                   (hipStream_t)stream);
}

int arn_policy_act(const arn_config *cfg, const void *w_packed, const uint8_t *obs, int B, const float *u,
                   const float *u2, float epsilon, int32_t *action, float *logp, void *workspace,
                   size_t workspace_bytes, void *stream) {
    if (!cfg || B <= 0 || B > (1 << 20)) return ARN_EINVAL;
    if (!known_head(cfg->head_kind)) return ARN_EKIND;
    const Dims d = make_dims(cfg);
    if (!d.ok) return ARN_ESHAPE;
    if (!aligned(w_packed, 256) || !aligned(obs, 16) || !aligned(u, 16) || !aligned(action, 16) ||
        !aligned(workspace, 256))
        return ARN_EINVAL;
    const bool policy = d.head == ARN_HEAD_PV;
    if (!policy && (!aligned(u2, 16) || !(epsilon >= 0.f && epsilon <= 1.f))) return ARN_EINVAL;
    if (logp && (!policy || !aligned(logp, 16))) return policy ? ARN_EINVAL : ARN_ESHAPE;
    const Workspace o = make_workspace(d, B, ARN_MODE_FORWARD);
    if (workspace_bytes < o.total) return ARN_EWORKSPACE;
    if (int e = check_arch()) return e;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    const Packed w = view_packed(w_packed, d);
    float *z = (float *)(ws + o.z);   // categorical head only
    PvHeadArgs p = pv_head_args(d, w, B, ws, o, 1);
    p.u = u; p.u2 = u2; p.epsilon = epsilon; p.act_out = action; p.logp_out = logp;
    infer_launches(d, w, obs, B, ws, o, z, d.NHP, &p, s);
    if (!d.small) {
        ProfScope ps("c51_dist", s);
        hipLaunchKernelGGL(c51_dist_kernel, dim3(cdiv(B, C51_WAVES)), dim3(64 * C51_WAVES), 0, s, z, d.NHP, B, d.A, d.atoms,
                           cfg->v_min, cfg->v_max, cfg->gamma, (const float *)nullptr, (const uint8_t *)nullptr,
                           (float *)nullptr, (float *)nullptr, action, (float *)nullptr);
        hipLaunchKernelGGL(epsilon_greedy_kernel, dim3(cdiv(B, 256)), dim3(256), 0, s, action, u, u2, epsilon, d.A, B);
    }
    return launched();
}

int arn_train_step_grads(const arn_config *cfg, const void *w_packed, const arn_batch *batch, int B, int loss_kind,
                         float *dW, float *loss, void *workspace, size_t workspace_bytes, void *stream) {
    if (!cfg || !batch || B <= 0 || B > (1 << 20)) return ARN_EINVAL;
    if (!known_head(cfg->head_kind)) return ARN_EKIND;
    if (loss_kind != ARN_LOSS_A2C && loss_kind != ARN_LOSS_PPO && loss_kind != ARN_LOSS_C51 &&
        loss_kind != ARN_LOSS_DQN)
        return ARN_EKIND;
    const Dims d = make_dims(cfg);
    if (!d.ok) return ARN_ESHAPE;
    if ((loss_kind == ARN_LOSS_C51) != (d.head == ARN_HEAD_C51)) return ARN_ESHAPE;
    if ((loss_kind == ARN_LOSS_DQN) != d.qhead) return ARN_ESHAPE;
    if (!aligned(w_packed, 256) || !aligned(batch->obs, 16) || !aligned(batch->action, 16) || !aligned(dW, 16) ||
        !aligned(loss, 16) || !aligned(workspace, 256))
        return ARN_EINVAL;
    if (loss_kind == ARN_LOSS_A2C || loss_kind == ARN_LOSS_PPO) {
        if (!aligned(batch->adv, 16) || !aligned(batch->ret, 16)) return ARN_EINVAL;
        if (loss_kind == ARN_LOSS_PPO && !aligned(batch->old_logp, 16)) return ARN_EINVAL;
    } else {
        if (!aligned(batch->next_obs, 16) || !aligned(batch->reward, 16) || !aligned(batch->done, 16) ||
            !aligned(batch->w_target_packed, 256))
            return ARN_EINVAL;
        if (batch->next_action && !aligned(batch->next_action, 16)) return ARN_EINVAL;
    }
    const Workspace o = make_workspace(d, B, ARN_MODE_TRAIN);
    if (workspace_bytes < o.total) return ARN_EWORKSPACE;
    if (int e = check_arch()) return e;

    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    const Packed w = view_packed(w_packed, d);
    float *z = (float *)(ws + o.z);
    __bf16 *h = (__bf16 *)(ws + o.h);
    __bf16 *dz = (__bf16 *)(ws + o.dz), *dph = (__bf16 *)(ws + o.dph);
    float *lossp = (float *)(ws + o.lossp), *hbp = (float *)(ws + o.hbp);
    const int lblocks = loss_blocks(d, B);
    // Double-DQN: the online network's greedy action on the next states, kept where the caller asked for it
    int32_t *const astar = batch->next_action ? batch->next_action : (int32_t *)(ws + o.astar);

    // ---- forward and objective ----
    // The passes that carry no gradient (target network, Double-DQN selection) are one fp16 product per layer.
    if (loss_kind == ARN_LOSS_C51) {
        // target network on next states -> projected target m; its activations are then overwritten
        const Packed wt = view_packed(batch->w_target_packed, d);
        float *ztgt = (float *)(ws + o.ztgt), *m = (float *)(ws + o.m);
        infer_launches(d, wt, batch->next_obs, B, ws, o, ztgt, d.NHP, nullptr, s);
        {
            ProfScope ps("c51_target", s);
            hipLaunchKernelGGL(c51_dist_kernel, dim3(cdiv(B, C51_WAVES)), dim3(64 * C51_WAVES), 0, s, ztgt, d.NHP, B, d.A,
                               d.atoms, cfg->v_min, cfg->v_max, cfg->gamma, batch->reward, batch->done,
                               (float *)nullptr, (float *)nullptr, batch->next_action, m);
        }
        forward_launches(d, w, batch->obs, B, ws, o, z, d.NHP, s);
        ProfScope ps("loss", s);
        hipLaunchKernelGGL(c51_loss_kernel, dim3(lblocks), dim3(64 * C51_WAVES), 0, s, z, d.NHP, m, batch->action, B, d.A,
                           d.atoms, d.NHP, c51_loss_spw(B), dz, lossp, hbp);
    } else {
        const Packed *wt = nullptr;
        Packed wt_view;
        if (loss_kind == ARN_LOSS_DQN) {
            // target network on the next states -> Q(s', .); with Double-DQN the online network on the next
            // states -> its greedy action.  The activations of these passes are then overwritten.
            wt_view = view_packed(batch->w_target_packed, d);
            wt = &wt_view;
            PvHeadArgs p = pv_head_args(d, *wt, B, ws, o, 1);
            p.logits = (float *)(ws + o.qt);
            if (!cfg->double_q) p.greedy = batch->next_action;
            infer_launches(d, *wt, batch->next_obs, B, ws, o, nullptr, 0, &p, s);
            if (cfg->double_q) {
                PvHeadArgs q = pv_head_args(d, w, B, ws, o, 1);
                q.greedy = astar;
                infer_launches(d, w, batch->next_obs, B, ws, o, nullptr, 0, &q, s);
            }
        }
        forward_launches(d, w, batch->obs, B, ws, o, nullptr, 0, s);
        // fc finish, head, objective, dz and the head's input gradient d(pre_fc) in one kernel
        ProfScope ps("pv_head", s);
        PvHeadArgs p = pv_head_args(d, w, B, ws, o, fc_ksplit(d.feat, d.hid, B, false));
        p.action = batch->action; p.adv = batch->adv; p.ret = batch->ret; p.old_logp = batch->old_logp;
        p.objective = loss_kind == ARN_LOSS_PPO ? 1 : loss_kind == ARN_LOSS_DQN ? 2 : 0;
        p.clip_eps = cfg->clip_eps; p.value_coef = cfg->value_coef; p.entropy_coef = cfg->entropy_coef;
        if (loss_kind == ARN_LOSS_DQN) {
            p.q_next = (const float *)(ws + o.qt);
            p.a_star = cfg->double_q ? astar : nullptr;
            p.reward = batch->reward; p.done = batch->done; p.gamma = cfg->gamma;
        }
        p.whd = w.whd; p.h = h; p.dz = dz; p.dph = dph; p.lossp = lossp; p.hbp = hbp;
        p.rpb = loss_block(B);
        if (d.hid == HID) hipLaunchKernelGGL((pv_head_kernel<true, HID>), dim3(lblocks), dim3(PVH_THREADS), 0, s, p);
        else hipLaunchKernelGGL((pv_head_kernel<true, GeoA3c::NHID>), dim3(lblocks), dim3(PVH_THREADS), 0, s, p);
    }

    // ---- backward ----
    const bool pv = loss_kind == ARN_LOSS_A2C || loss_kind == ARN_LOSS_PPO;
    const LossTotals totals{lossp, lblocks, B, pv ? cfg->value_coef : 0.f, pv ? cfg->entropy_coef : 0.f, loss};
    with_geometry(d, [&](auto g) {
        typedef decltype(g) G;
        if (d.head == ARN_HEAD_C51) {
            with_tile(B, G::NHID, [&](auto bm) {
                HeadDgrad<G::NHID, decltype(bm)::value> p;
                p.in = dz; p.M = B; p.K = d.NHP; p.w = w.whd; p.h = h; p.out = dph;
                launch_nt<false>("head_dgrad", p, G::NHID, 1, s);
            });
        }
        backward_trunk<G>(d, w, batch->obs, B, ws, o, totals, lblocks, dW, s);
    });
    return launched();
}

int arn_rmsprop_update(size_t n, float *theta, const float *g, float *accu, float lr, float rho, float eps,
                       const arn_config *cfg, void *w_packed, void *stream) {
    bool repack;
    Dims d;
    if (int e = check_update(n, cfg, w_packed, &repack, &d)) return e;
    if (!aligned(theta, 16) || !aligned(g, 16) || !aligned(accu, 16)) return ARN_EINVAL;
    if (!unit_interval(rho) || !(eps >= 0.f) || !(lr == lr)) return ARN_EINVAL;
    if (int e = check_arch()) return e;
    hipStream_t s = (hipStream_t)stream;
    UpdateArgs p = {};
    p.theta = theta; p.g = g; p.v = accu; p.n = (long)n; p.a = lr; p.beta2 = rho; p.eps = eps;
    launch_update<RULE_RMSPROP>("rmsprop", p, repack, d, w_packed, s);
    return launched();
}

namespace {
// a = r sqrt(1 - beta2^t) / (1 - beta1^t), formed in fp64
float adam_scale(int64_t t, float r, float beta1, float beta2) {
    const double c1 = 1.0 - pow((double)beta1, (double)t), c2 = 1.0 - pow((double)beta2, (double)t);
    return (float)((double)r * sqrt(c2) / c1);
}
}  // namespace

int arn_adam_update(size_t n, float *theta, const float *g, float *m, float *v, int64_t t, float r, float beta1,
                    float beta2, float eps, const arn_config *cfg, void *w_packed, void *stream) {
    bool repack;
    Dims d;
    if (int e = check_update(n, cfg, w_packed, &repack, &d)) return e;
    if (!aligned(theta, 16) || !aligned(g, 16) || !aligned(m, 16) || !aligned(v, 16)) return ARN_EINVAL;
    if (t < 1 || !unit_interval(beta1) || !unit_interval(beta2) || !(eps >= 0.f) || !(r == r)) return ARN_EINVAL;
    if (int e = check_arch()) return e;
    hipStream_t s = (hipStream_t)stream;
    UpdateArgs p = {};
    p.theta = theta; p.g = g; p.m = m; p.v = v; p.n = (long)n;
    p.a = adam_scale(t, r, beta1, beta2); p.beta1 = beta1; p.beta2 = beta2; p.eps = eps;
    launch_update<RULE_ADAM>("adam", p, repack, d, w_packed, s);
    return launched();
}

int arn_async_adam_local_step(size_t n, float *theta, const float *g, float *m, float *v, float *a_g, float *a_g2,
                              float *a_s, int64_t t, float r, float beta1, float beta2, float eps,
                              const arn_config *cfg, void *w_packed, void *stream) {
    bool repack;
    Dims d;
    if (int e = check_update(n, cfg, w_packed, &repack, &d)) return e;
    if (!aligned(theta, 16) || !aligned(g, 16) || !aligned(m, 16) || !aligned(v, 16) || !aligned(a_g, 16) ||
        !aligned(a_g2, 16) || !aligned(a_s, 16))
        return ARN_EINVAL;
    if (t < 1 || !unit_interval(beta1) || !unit_interval(beta2) || !(eps >= 0.f) || !(r == r)) return ARN_EINVAL;
    if (int e = check_arch()) return e;
    hipStream_t s = (hipStream_t)stream;
    UpdateArgs p = {};
    p.theta = theta; p.g = g; p.m = m; p.v = v; p.a_g = a_g; p.a_g2 = a_g2; p.a_s = a_s; p.n = (long)n;
    p.a = adam_scale(t, r, beta1, beta2); p.beta1 = beta1; p.beta2 = beta2; p.eps = eps;
    launch_update<RULE_ADAM_LOCAL>("adam_local", p, repack, d, w_packed, s);
    return launched();
}

int arn_async_adam_merge(size_t n, float *theta_c, float *m_c, float *v_c, float *theta, float *m, float *v,
                         float *a_g, float *a_g2, float *a_s, int n_local, float beta1, float beta2,
                         const arn_config *cfg, void *w_packed, void *stream) {
    bool repack;
    Dims d;
    if (int e = check_update(n, cfg, w_packed, &repack, &d)) return e;
    if (!aligned(theta_c, 16) || !aligned(m_c, 16) || !aligned(v_c, 16) || !aligned(theta, 16) || !aligned(m, 16) ||
        !aligned(v, 16) || !aligned(a_g, 16) || !aligned(a_g2, 16) || !aligned(a_s, 16))
        return ARN_EINVAL;
    if (theta_c == theta || m_c == m || v_c == v) return ARN_EINVAL;
    if (n_local < 0 || !unit_interval(beta1) || !unit_interval(beta2)) return ARN_EINVAL;
    if (int e = check_arch()) return e;
    hipStream_t s = (hipStream_t)stream;
    UpdateArgs p = {};
    p.theta_c = theta_c; p.m_c = m_c; p.v_c = v_c; p.theta = theta; p.m = m; p.v = v;
    p.a_g = a_g; p.a_g2 = a_g2; p.a_s = a_s; p.n = (long)n; p.beta1 = beta1; p.beta2 = beta2;
    p.beta1_n = (float)pow((double)beta1, (double)n_local);
    p.beta2_n = (float)pow((double)beta2, (double)n_local);
    launch_update<RULE_MERGE>("adam_merge", p, repack, d, w_packed, s);
    return launched();
}

int arn_profile_null(void *stream) {
    // an event pair around nothing: what the instrumentation itself adds to every recorded duration
    ProfScope ps("null", (hipStream_t)stream);
    return ARN_OK;
}

int arn_profile_enable(int on) {
    g_prof_on = on != 0;
    return ARN_OK;
}

int arn_profile_collect(char *names, float *ms, int cap) {
    int n = 0;
    for (const ProfRecord &r : g_prof) {
        float t = 0.f;
        if (r.stop && hipEventSynchronize(r.stop) == hipSuccess) (void)hipEventElapsedTime(&t, r.start, r.stop);
        if (n < cap && names && ms) {
            strncpy(names + (size_t)n * 32, r.name, 31);
            names[(size_t)n * 32 + 31] = 0;
            ms[n] = t;
            ++n;
        }
        if (r.start) (void)hipEventDestroy(r.start);
        if (r.stop) (void)hipEventDestroy(r.stop);
    }
    g_prof.clear();
    return n;
}

}  // extern "C"
