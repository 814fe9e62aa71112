"""GPU parity where the small-batch kernels hand over: sizes on both sides of every tile and dispatch edge of the banded
convolutions and of fc_small_kernel, against the CPU oracle (the bars of tests/gpu_util.py)."""
import numpy as np
import pytest

import workloads as wl
from oracle import nature_cnn as orc

pytestmark = pytest.mark.gpu
NETS = {"84": (wl.FRAME, {}), "paper": (wl.PAPER_FRAME, {"geometry": orc.PAPER_104x80}),
        "a3c": (wl.PAPER_FRAME, {"geometry": orc.A3C_104x80})}


def shape_of(geometry):
    return dict(net="a3c") if geometry == "a3c" else dict(fc_inputs=wl.FC_INPUTS[NETS[geometry][0]])


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("geometry,head,sizes", [
    ("84", "pv", (17, 32, 36, 37, 63, 65, 127, 128, 129, 255, 257, 511, 512, 513)),
    ("84", "c51", (33, 129, 513)),
    ("paper", "duel", (21, 22, 65, 86, 128, 129, 257, 361, 362)),
    ("a3c", "pv", (21, 22, 33, 64, 127, 128, 129, 256, 257, 512, 513)),
    ("a3c", "c51", (40, 513))])
def test_forward_at_dispatch_edges(gu, geometry, head, sizes):
    A = 7
    frame, kw = NETS[geometry]
    flat = wl.he_normal_params(A, head, 2602, bias_std=0.1, **shape_of(geometry))
    spec = orc.NetSpec(A, head, **kw)
    obs = wl.rect_frames(max(sizes), 1602, frame=frame)
    ref = orc.forward(orc.unflatten(flat, spec), obs, spec)
    want = ref[{"pv": "logits", "duel": "q", "c51": "atom_logits"}[head]]
    net = gu.GpuNet(A, head, flat, geometry=geometry)
    for B in sizes:
        out = net.forward(obs[:B])
        got = out["q" if head == "duel" else "logits"]
        gu.tol_check(got, want[:B].reshape(got.shape), "B=%d" % B)


@pytest.mark.parametrize("geometry,B", [("84", 129), ("84", 398), ("84", 399), ("84", 641), ("84", 1281), ("paper", 65), ("paper", 180), ("paper", 181),
                                        ("a3c", 21), ("a3c", 128), ("a3c", 129), ("a3c", 361), ("a3c", 362)])
def test_gradients_at_dispatch_edges(gu, geometry, B):
    A = 7
    frame, kw = NETS[geometry]
    flat = wl.he_normal_params(A, "pv", 2603, bias_std=0.1, **shape_of(geometry))
    batch = wl.actor_critic_batch(3, B=B, frame=frame)
    batch["action"] %= A
    ref = orc.train_step_grads(flat, batch, "a2c", orc.NetSpec(A, "pv", **kw))
    dW, _ = gu.GpuNet(A, "pv", flat, geometry=geometry).train(batch, "a2c")
    got, want = (wl.split_params(v, A, "pv", **shape_of(geometry)) for v in (dW, ref["flat"]))
    gu.check_grads(got, want, "%s B=%d" % (geometry, B))


@pytest.mark.parametrize("geometry,B", [("84", 1280), ("84", 2432), ("84", 2433), ("84", 2463), ("paper", 1152), ("paper", 1153)])
def test_gradients_at_fc_weight_tile_edges(gu, geometry, B):
    """Both sides of the batch from which the fc weight gradient takes 256 hidden units a tile (84x84: 2433, 104x80: 1153) and of the
    one from which the input gradient takes 128 positions (84x84: 1281), last stages of 1, 31 and 32 rows."""
    test_gradients_at_dispatch_edges(gu, geometry, B)


@pytest.mark.parametrize("B", [64, 257])
def test_gradients_at_chained_convolution_edges(gu, B):
    """104x80: the last batch with a launch per convolution (from 65 on they are one), and two samples a workgroup with one left over."""
    test_gradients_at_dispatch_edges(gu, "paper", B)


# padded head rows 64 (fewer stages than the dense kernel has slots), 192 and 960 (the last tile half full)
@pytest.mark.parametrize("A,B", [(1, 33), (3, 129), (18, 70)])
def test_categorical_gradients_at_tile_edges(gu, A, B):
    flat, tflat = (wl.he_normal_params(A, "c51", seed, bias_std=0.1) for seed in (2615, 3615))
    batch = wl.c51_batch(5, B=B)
    batch["action"] %= A
    dW, _, ref, _ = gu.train_c51_or_dqn(gu.GpuNet(A, "c51", flat), orc, flat, tflat, batch, "c51", orc.NetSpec(A, "c51"))
    got, want = (wl.split_params(v, A, "c51") for v in (dW, ref["flat"]))
    gu.check_grads(got, want, "A=%d B=%d" % (A, B))


# 84x84: the last batch whose fc contraction is cut in two and the first whose is not: its tiles write the hidden layer themselves
@pytest.mark.parametrize("B", [4096, 4097])
def test_categorical_network_where_the_fc_tiles_finish_the_layer(gu, B):
    """Logits of the first and last samples against the oracle; the gradient against the mean of two shards, whose contraction is
    cut.  One action, so that no greedy decision stands between them."""
    A = 1
    flat, tflat = (wl.he_normal_params(A, "c51", seed, bias_std=0.1) for seed in (2618, 3618))
    batch = wl.c51_batch(5, B=B)
    batch["action"] %= A
    net, spec = gu.GpuNet(A, "c51", flat), orc.NetSpec(A, "c51")
    rows = np.r_[0:9, B - 9:B]
    want = orc.forward(orc.unflatten(flat, spec), batch["obs"][rows], spec)["atom_logits"]
    got = net.forward(batch["obs"])["logits"][rows]
    gu.tol_check(got, want.reshape(got.shape), "B=%d" % B)
    target = net.pack(tflat)
    whole = net.train(batch, "c51", target_packed=target)[0]
    shards = [slice(0, 2048), slice(2048, B)]
    mean = sum((s.stop - s.start) / B * net.train({k: v[s] for k, v in batch.items()}, "c51", target_packed=target)[0].astype(np.float64)
               for s in shards)
    gu.check_grads(*(wl.split_params(v, A, "c51") for v in (whole, mean)), "B=%d against two shards" % B)


# Batches whose passes without gradient run in fc_small_kernel (activations in fragment order) while the forward pass of the
# same step, in the same workspace, runs in the tiled GEMM (activations in rows, several k ranges): both ends of that window.
@pytest.mark.parametrize("geometry,head,B", [("84", "duel", 399), ("84", "q", 512), ("84", "c51", 450),
                                             ("paper", "duel", 181), ("paper", "q", 361), ("paper", "c51", 300),
                                             ("a3c", "duel", 362), ("a3c", "c51", 512)])
def test_bootstrapped_gradients_where_both_dense_paths_meet(gu, geometry, head, B):
    A = 7
    frame, kw = NETS[geometry]
    kind, double_q = ("c51", 0) if head == "c51" else ("dqn", int(head == "duel"))
    flat, tflat = (wl.he_normal_params(A, head, seed, bias_std=0.1, **shape_of(geometry)) for seed in (2617, 3617))
    batch = wl.c51_batch(5, B=B, frame=frame)
    batch["action"] %= A
    net = gu.GpuNet(A, head, flat, geometry=geometry, double_q=double_q)
    net.workspace(B, 1).fill_(255)                 # whatever the workspace holds (here: not-a-numbers)
    hyper = orc.Hyper(double_q=True) if double_q else None
    dW, _, ref, _ = gu.train_c51_or_dqn(net, orc, flat, tflat, batch, kind, orc.NetSpec(A, head, **kw), hyper=hyper)
    got, want = (wl.split_params(v, A, head, **shape_of(geometry)) for v in (dW, ref["flat"]))
    gu.check_grads(got, want, "%s %s B=%d" % (geometry, head, B))


# sizes on each side of the edges between bands and whole samples and between the tiles of fc_small_kernel, up to its largest
@pytest.mark.parametrize("geometry,head,sizes", [
    ("84", "pv", (1, 17, 36, 37, 64, 65, 128, 129, 256, 257, 512)),
    ("84", "c51", (1, 17, 37, 129, 300, 512)),
    ("paper", "duel", (1, 17, 21, 22, 64, 65, 129, 257, 361)),
    ("a3c", "pv", (1, 17, 21, 22, 128, 129, 257, 512))])
def test_outputs_do_not_depend_on_the_batch(gu, geometry, head, sizes):
    """A sample's outputs have the same bits in every batch that fc_small_kernel serves, whatever the workspace holds."""
    A = 7
    flat = wl.he_normal_params(A, head, 2602, bias_std=0.1, **shape_of(geometry))
    obs = wl.rect_frames(max(sizes), 1602, frame=NETS[geometry][0])
    net = gu.GpuNet(A, head, flat, geometry=geometry)
    whole = net.forward(obs)
    for B in sizes:
        net.workspace(B, 0).fill_(255)
        for name, got in net.forward(obs[:B]).items():
            assert np.array_equal(got, whole[name][:B]), (name, B)
