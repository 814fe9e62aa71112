"""bench.py's counter summaries: every kernel is booked under its own launch name, and figures of replaced kernels are not
reported."""
import json
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1803_02811_amd", "csrc")
GEO84 = "arn::Geometry<84, 84, 0, 0, 32, 64, true, 512>"
# kernel -> names as rocprofv3 prints them (demangled, or mangled where it does not know a type) and their launch names
NAMES = {
    "conv123_fwd_kernel": [("_ZN3arn18conv123_fwd_kernelINS_8GeometryILi84ELi84ELi0ELi0ELi32ELi64ELb1ELi512EEENS_11ResConv2FwdENS_11ResConv3FwdEEEvPKh",
                            "conv123_fwd")],
    "conv123_chain_kernel": [("_ZN3arn20conv123_chain_kernelINS_8GeometryILi104ELi80ELi1ELi1ELi32ELi64ELb1ELi512EEENS_14ResConv2FwdGeoIS2_EE", "conv123_fwd")],
    "conv23_fwd_fused_kernel": [("void arn::conv23_fwd_fused_kernel<arn::ResConv2Fwd, arn::ResConv3Fwd>(arn::Conv23Args, int, int)", "conv23_fwd")],
    "conv12_fwd_kernel": [("void arn::conv12_fwd_kernel<G, arn::ResConv2FwdGeo<G> >(arn::Conv12Args, int, int, int, int)", "conv12_fwd")],
    "conv1_fwd_resident_kernel": [("void arn::conv1_fwd_resident_kernel<%s >(unsigned char const*)" % GEO84, "conv1_fwd")],
    "infer_conv_kernel": [("void arn::infer_conv_kernel<G, arn::ResConv2FwdGeo<G>, arn::NoConv3, true>(arn::InferConvArgs, int, int)", "conv_infer")],
    "infer_conv_pipelined_kernel": [("void arn::infer_conv_pipelined_kernel<%s, arn::ResConv2Fwd, arn::ResConv3Fwd, true>(arn::InferConvArgs, int, int)" % GEO84,
                                     "conv_infer")],
    "infer_conv_band_kernel": [("void arn::infer_conv_band_kernel<%s, arn::ResConv2Fwd, arn::ResConv3Fwd>(arn::InferConvArgs, int, int)" % GEO84, "conv_infer")],
    "conv_backward_kernel": [("void arn::conv_backward_kernel<%s, arn::ResConv2Dgrad>(arn::ConvBackwardArgs)" % GEO84, "conv_bwd")],
    "dense_backward_kernel": [("void arn::dense_backward_kernel<arn::FcDgradT<3136, 512, 64>, arn::FcWgrad<3136, 512>, arn::HeadWgrad<512> >()", "dense_bwd")],
    "reduce_all_kernel": [("void arn::reduce_all_kernel<%s >(arn::ReduceAllPlan<%s >, float*)" % (GEO84, GEO84), "reduce")],
    "resident_conv_kernel": [("void arn::resident_conv_kernel<arn::ResConv2Fwd>(arn::ResConv2Fwd::Args, int, int)", "conv2_fwd"),
                             ("void arn::resident_conv_kernel<arn::ResConv3FwdGeo<G> >()", "conv3_fwd"),
                             ("void arn::resident_conv_kernel<arn::ResConv3DgradGeo<G> >()", "conv3_dgrad")],
    "gemm_nt_kernel": [("void arn::gemm_nt_kernel<arn::FcFwdT<3136, 512, 128>, true>(arn::FcFwdT<3136, 512, 128>)", "fc_fwd"),
                       ("void arn::gemm_nt_kernel<arn::FcFwdF16T<6912, 512, 64>, false>()", "fc_fwd"),
                       ("void arn::gemm_nt_kernel<arn::HeadFwdC51<512, 64>, true>()", "head_fwd"),
                       ("void arn::gemm_nt_kernel<arn::HeadDgrad<512, 64>, false>()", "head_dgrad")],
    "fc_small_kernel": [("void arn::fc_small_kernel<3136, 512, 2, 2, true, 2>(arn::FcSmallArgs)", "fc_head"),
                        ("_ZN3arn15fc_small_kernelILi3456ELi256ELi1ELi1ELb1ELi2EEEvNS_11FcSmallArgsE", "fc_head"),
                        ("void arn::fc_small_kernel<3136, 512, 2, 2, true, 1>(arn::FcSmallArgs)", "fc_fwd"),
                        ("_ZN3arn15fc_small_kernelILi3136ELi512ELi2ELi2ELb0ELi0EEEvNS_11FcSmallArgsE", "fc_fwd")],
    "pv_head_kernel": [("void arn::pv_head_kernel<true, 512>(arn::PvHeadArgs)", "pv_head"),
                       ("_ZN3arn14pv_head_kernelILb1ELi256EEEvNS_10PvHeadArgsE", "pv_head"),
                       ("void arn::pv_head_kernel<false, 256>(arn::PvHeadArgs)", "pv_head_infer")],
    "fc_finish_kernel": [("arn::fc_finish_kernel(float const*, int, float const*, __bf16*, __bf16*, int, long)", "fc_finish")],
    "c51_dist_kernel": [("arn::c51_dist_kernel(float const*, int)", "c51_dist")],
    "c51_loss_kernel": [("_ZN3arn15c51_loss_kernelEPKfiS1_PKiiiiiiPDF16bPfS5_", "loss")],
    "update_kernel": [("void arn::update_kernel<0>(arn::UpdateArgs)", "rmsprop"), ("void arn::update_kernel<2>(arn::UpdateArgs)", "adam_local")],
    "update_pack_kernel": [("void arn::update_pack_kernel<1, %s >(arn::PackPlan<%s >, arn::UpdateArgs)" % (GEO84, GEO84), "adam"),
                           ("_ZN3arn18update_pack_kernelILi3ENS_8GeometryILi84ELi84E", "adam_merge")],
    "epsilon_greedy_kernel": [("arn::epsilon_greedy_kernel(int*, float const*)", "epsilon_greedy")],
    "pack_all_kernel": [("void arn::pack_all_kernel<%s >(arn::PackPlan<%s >, float const*)" % (GEO84, GEO84), "pack_all")],
}


def test_every_kernel_is_booked_under_its_launch_name():
    kernels = set()
    for f in os.listdir(CSRC):
        text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())
        kernels |= set(re.findall(r"__global__[^;{]*?\b(\w+_kernel)\s*\(", text))
    assert kernels == set(NAMES)
    for names in NAMES.values():
        for name, want in names:
            assert bench._short_kernel_name(name) == want, name


def test_traffic_of_other_kernels_is_not_reported(tmp_path, monkeypatch):
    """A summary names the sources that it was measured on: its figures are reported for these alone."""
    csrc = tmp_path / "paper_1803_02811_amd" / "csrc"
    csrc.mkdir(parents=True)
    (tmp_path / "profiles").mkdir()
    source = csrc / "k.h"
    source.write_text("int f() { return 1; }\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    summary = {"kernel_sources": bench.kernel_sources_digest(), "hbm_bytes_per_launch": {"conv_infer": 7}}
    (tmp_path / "profiles" / "w_traffic.json").write_text(json.dumps(summary))
    assert bench.measured_traffic("conv_infer", "w") == 7
    source.write_text("// measured\nint f() { /* one */ return 1; }\n")
    assert bench.measured_traffic("conv_infer", "w") == 7
    source.write_text("int f() { return 2; }\n")
    assert bench.measured_traffic("conv_infer", "w") is None
