"""The work a user of this library has it do, as cases that can be timed: batched action selection for a sampler,
evaluation of whole rollouts, gradient steps of the four objectives, learner iterations (gradient, update rule, re-pack)
and parameter updates, on the three networks (84x84 frames, the paper's 104x80 frames, the paper's 2-convolution
policy-gradient network).

Sizes are those of workloads.py (16, 256, 2048, 4096, 8192 samples), of the paper's own runs (16 environments x 5 steps,
replay batches of 512, groups of 128 simulators) and ragged ones between them.  All inputs are seeded and made on the GPU.
"""
import math

import torch

import paper_1803_02811_amd as arn

FRAME = {"84": (84, 84), "paper": (104, 80), "a3c": (104, 80)}
# (input channels, filters, kernel, output positions) of the convolutions; (inputs, units) of the fc layer
CONVS = {
    "84": [(4, 32, 8, 20 * 20), (32, 64, 4, 9 * 9), (64, 64, 3, 7 * 7)],
    "paper": [(4, 32, 8, 25 * 19), (32, 64, 4, 12 * 9), (64, 64, 3, 12 * 9)],
    "a3c": [(4, 16, 8, 25 * 19), (16, 32, 4, 12 * 9)],
}
FC = {"84": (3136, 512), "paper": (6912, 512), "a3c": (3456, 256)}
ATOMS = 51
OBJECTIVE_HEAD = {"a2c": "pv", "ppo": "pv", "c51": "c51", "dqn": "duel"}
# fp32 state arrays that each update rule reads and writes per parameter (theta, gradient, moments, accumulators)
UPDATE_BYTES = {"rmsprop": 20, "adam": 28, "async": 52, "merge": 60}


def listed():
    return [
        # a small sampler: one observation of each of 16 simulators, 6 actions; latency is everything
        dict(name="forward_b16", kind="forward", geometry="84", head="pv", actions=6, batch=16),
        # action selection over 256 simulators with the full action set: probabilities, greedy actions, values
        dict(name="forward_b256", kind="forward", geometry="84", head="pv", actions=18, batch=256),
        # evaluating a whole rollout (values for bootstrapping, probabilities) of 256 simulators x 8 steps
        dict(name="forward_b2048", kind="forward", geometry="84", head="pv", actions=18, batch=2048),
        # the paper's sampler: one of two alternating groups of simulators, actions and log-probabilities drawn
        dict(name="act_a3c_b128", kind="act", geometry="a3c", head="pv", actions=6, batch=128),
        # epsilon-greedy action selection of the value-based agents on the paper's frames, a ragged group
        dict(name="act_duel_paper_b75", kind="act", geometry="paper", head="duel", actions=9, batch=75),
        # the smallest gradient step in use: 16 environments x 5 steps on the policy-gradient network
        dict(name="a2c_a3c_b80", kind="train", geometry="a3c", objective="a2c", actions=6, batch=80),
        # a learner's iteration at a ragged batch: gradient, RMSProp, re-pack of the weights
        dict(name="learn_a2c_b333", kind="learn", geometry="84", objective="a2c", actions=18, batch=333),
        # Double-DQN with the dueling head at the paper's replay batch on the paper's frames
        dict(name="dqn_paper_b512", kind="train", geometry="paper", objective="dqn", actions=18, batch=512),
        # 256 environments x 8 steps: the headline gradient step
        dict(name="a2c_b2048", kind="train", geometry="84", objective="a2c", actions=18, batch=2048),
        # a PPO minibatch
        dict(name="ppo_b4096", kind="train", geometry="84", objective="ppo", actions=18, batch=4096),
        # the paper's largest batches: categorical DQN, target network included
        dict(name="c51_b8192", kind="train", geometry="84", objective="c51", actions=18, batch=8192),
        # Adam on a categorical network's parameters with the re-pack, what follows every such gradient
        dict(name="adam_c51", kind="update", geometry="84", head="c51", actions=18, rule="adam"),
    ]


def draw(rng):
    def log_uniform(lo, hi):
        return min(hi, int(lo * (hi / lo + 1e-9) ** rng.random() + 0.5))

    kind = rng.choice(["forward", "act", "train", "train", "train", "learn", "update"])
    geometry = rng.choice(["84", "84", "paper", "a3c"])
    case = dict(kind=kind, geometry=geometry, actions=rng.choice([4, 6, 9, 18]))
    if kind in ("forward", "act"):
        case.update(head=rng.choice(["pv", "pv", "duel", "q", "c51"]), batch=log_uniform(1, 4096))
    elif kind == "train":
        case.update(objective=rng.choice(["a2c", "ppo", "dqn", "c51"]), batch=log_uniform(16, 4096))
        if geometry == "84" and case["objective"] in ("a2c", "ppo"):
            case["batch"] = log_uniform(16, 8192)
    elif kind == "learn":
        case.update(objective="a2c", batch=log_uniform(16, 4096))
    else:
        case.update(head=rng.choice(["pv", "duel", "c51"]), rule=rng.choice(["rmsprop", "adam", "async", "merge"]),
                    actions=rng.randint(3, 18))
    return case


def head_of(case):
    return case.get("head") or OBJECTIVE_HEAD[case["objective"]]


def head_rows(case):
    """Rows of the head's weight matrix."""
    return {"pv": case["actions"] + 1, "duel": case["actions"] + 1, "q": case["actions"],
            "c51": case["actions"] * ATOMS}[head_of(case)]


def config(case):
    return arn.Config(num_actions=case["actions"], head_kind=arn.HEAD_KINDS[head_of(case)], num_atoms=ATOMS,
                      double_q=1 if case.get("objective") == "dqn" else 0, geometry=arn.GEOMETRIES[case["geometry"]])


# ---- inputs -------------------------------------------------------------------------------------------------------

def frame_stacks(count, batch, height, width, gen):
    """`count` consecutive observations of each of `batch` simulators, uint8 [batch,4,height,width]: black background,
    4 to 12 rectangles of side 4..32 and intensity 1..255, the scene moving by 1..3 pixels a frame in each direction."""
    def ints(lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=gen, device="cuda")

    ys, xs = torch.arange(height, device="cuda"), torch.arange(width, device="cuda")
    base = torch.zeros(batch, height, width, dtype=torch.uint8, device="cuda")
    number = ints(4, 13, batch)
    for k in range(12):
        h, w = ints(4, 33, batch), ints(4, 33, batch)
        top, left = ints(0, 1 << 20, batch) % (height - h + 1), ints(0, 1 << 20, batch) % (width - w + 1)
        rows = (ys >= top[:, None]) & (ys < (top + h)[:, None]) & (k < number)[:, None]
        cols = (xs >= left[:, None]) & (xs < (left + w)[:, None])
        value = ints(1, 256, batch).to(torch.uint8)
        base = torch.where(rows[:, :, None] & cols[:, None, :], value[:, None, None], base)
    dy = ints(1, 4, batch) * (2 * ints(0, 2, batch) - 1)
    dx = ints(1, 4, batch) * (2 * ints(0, 2, batch) - 1)
    frames = []
    for f in range(3 + count):
        y, x = ys - f * dy[:, None], xs - f * dx[:, None]
        inside = ((y >= 0) & (y < height))[:, :, None] & ((x >= 0) & (x < width))[:, None, :]
        at = y.clamp(0, height - 1)[:, :, None] * width + x.clamp(0, width - 1)[:, None, :]
        moved = base.view(batch, -1).gather(1, at.view(batch, -1)).view(batch, height, width)
        frames.append(moved * inside)
    return [torch.stack(frames[i:i + 4], 1) for i in range(count)]


def parameters(case, gen):
    """He-normal weights and zero biases as one flat fp32 vector.  PPO starts from a nearly uniform policy (its
    policy head is initialised a hundred times smaller), which is what the old log-probabilities below belong to."""
    parts = []

    def layer(fan_in, units, scale=1.0):
        parts.append(torch.randn(units * fan_in, generator=gen, device="cuda") * (scale * math.sqrt(2.0 / fan_in)))
        parts.append(torch.zeros(units, device="cuda"))

    for cin, cout, k, _ in CONVS[case["geometry"]]:
        layer(cin * k * k, cout)
    inputs, hidden = FC[case["geometry"]]
    layer(inputs, hidden)
    if head_of(case) in ("pv", "duel"):
        layer(hidden, case["actions"], 0.01 if case.get("objective") == "ppo" else 1.0)
        layer(hidden, 1)
    else:
        layer(hidden, head_rows(case))
    return torch.cat(parts)


def packed(cfg, theta):
    blob = torch.empty(arn.packed_bytes(cfg), dtype=torch.uint8, device="cuda")
    arn.weights_prepare(cfg, theta, blob)
    return blob


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cfg, kind, batch = config(case), case["kind"], case.get("batch")
    s = dict(case=case, cfg=cfg)
    theta = parameters(case, gen)
    assert theta.numel() == arn.param_count(cfg)
    s["packed"] = packed(cfg, theta)
    if kind == "update":
        prepare_update(s, theta, gen)
        return s
    mode = arn.ARN_MODE_FORWARD if kind in ("forward", "act") else arn.ARN_MODE_TRAIN
    s["workspace"] = torch.empty(arn.workspace_bytes(cfg, batch, mode), dtype=torch.uint8, device="cuda")
    if kind in ("forward", "act"):
        prepare_inference(s, batch, gen)
    else:
        prepare_training(s, batch, gen)
    if kind == "learn":
        s["theta"], s["accu"] = theta, torch.zeros_like(theta)
    return s


def prepare_inference(s, batch, gen):
    case, head, actions = s["case"], head_of(s["case"]), s["case"]["actions"]
    s["obs"], = frame_stacks(1, batch, *FRAME[case["geometry"]], gen)
    f32 = dict(dtype=torch.float32, device="cuda")
    if case["kind"] == "act":
        s["u"], s["u2"] = torch.rand(batch, generator=gen, **f32), torch.rand(batch, generator=gen, **f32)
        s["out"] = dict(action=torch.empty(batch, dtype=torch.int32, device="cuda"))
        if head == "pv":
            s["out"]["logp"] = torch.empty(batch, **f32)
        return
    s["out"] = dict(logits=torch.empty(batch, head_rows(case) if head == "c51" else actions, **f32),
                    value=torch.empty((batch, actions) if head == "c51" else (batch,), **f32),
                    greedy=torch.empty(batch, dtype=torch.int32, device="cuda"))
    if head == "pv":
        s["out"]["probs"] = torch.empty(batch, actions, **f32)


def prepare_training(s, batch, gen):
    case, cfg, actions, objective = s["case"], s["cfg"], s["case"]["actions"], s["case"]["objective"]
    f32 = dict(dtype=torch.float32, device="cuda")
    b = dict(action=torch.randint(0, actions, (batch,), generator=gen, dtype=torch.int32, device="cuda"))
    if objective in ("a2c", "ppo"):
        b["obs"], = frame_stacks(1, batch, *FRAME[case["geometry"]], gen)
        b["adv"] = torch.randn(batch, generator=gen, **f32)
        b["ret"] = torch.randn(batch, generator=gen, **f32)
        if objective == "ppo":
            b["adv"] = (b["adv"] - b["adv"].mean()) / (b["adv"].std(unbiased=False) + 1e-8)
            b["old_logp"] = 0.05 * torch.randn(batch, generator=gen, **f32) - math.log(actions)
    else:
        b["obs"], b["next_obs"] = frame_stacks(2, batch, *FRAME[case["geometry"]], gen)
        b["reward"] = torch.randint(-1, 2, (batch,), generator=gen, device="cuda").float()
        b["done"] = (torch.rand(batch, generator=gen, device="cuda") < 0.01).to(torch.uint8)
        b["w_target_packed"] = packed(cfg, parameters(case, gen))
        b["next_action"] = torch.empty(batch, dtype=torch.int32, device="cuda")
    s["batch"] = b
    s["dW"] = torch.empty(arn.param_count(cfg), **f32)
    s["loss"] = torch.empty(4, **f32)


def prepare_update(s, theta, gen):
    n, rule = theta.numel(), s["case"]["rule"]

    def gradient():
        """Entries whose magnitudes spread over decades, as across the layers of a deep network; some exactly zero."""
        g = torch.randn(n, generator=gen, device="cuda") * 10.0 ** (5 * torch.rand(n, generator=gen, device="cuda") - 6)
        return g * (torch.rand(n, generator=gen, device="cuda") > 0.01)

    # moments as a few steps leave them
    s.update(theta=theta, g=gradient(), m=gradient() * 0.1, v=gradient().square() * 0.1, t=10)
    if rule in ("async", "merge"):
        s.update(a_g=gradient(), a_g2=gradient().square(), a_s=gradient() * 1e-2)
    if rule == "merge":
        s.update(theta_c=theta + 1e-3 * gradient(), m_c=gradient() * 0.1, v_c=gradient().square() * 0.1)


# ---- one pass -----------------------------------------------------------------------------------------------------

def run(s):
    case, cfg, kind = s["case"], s["cfg"], s["case"]["kind"]
    if kind == "forward":
        arn.policy_forward(cfg, s["packed"], s["obs"], **s["out"], workspace=s["workspace"])
        return s["out"]
    if kind == "act":
        arn.policy_act(cfg, s["packed"], s["obs"], s["u"], s["u2"], **s["out"], epsilon=0.1, workspace=s["workspace"])
        return s["out"]
    if kind == "update":
        return run_update(s, case["rule"])
    arn.train_step_grads(cfg, s["packed"], s["batch"], case["objective"], s["dW"], s["loss"], workspace=s["workspace"])
    out = dict(dW=s["dW"], loss=s["loss"])
    if "next_action" in s["batch"]:
        out["next_action"] = s["batch"]["next_action"]
    if kind == "learn":
        arn.rmsprop_update(s["theta"], s["dW"], s["accu"], lr=1e-4, rho=0.99, eps=1e-5, cfg=cfg, w_packed=s["packed"])
        out.update(theta=s["theta"], accu=s["accu"])
    return out


def run_update(s, rule):
    pack = dict(cfg=s["cfg"], w_packed=s["packed"])
    adam = dict(r=1e-4, beta1=0.9, beta2=0.999, eps=1e-4)
    s["t"] += 1
    if rule == "rmsprop":
        arn.rmsprop_update(s["theta"], s["g"], s["v"], lr=1e-4, rho=0.99, eps=1e-5, **pack)
        return [s[k] for k in ("theta", "v")]
    if rule == "adam":
        arn.adam_update(s["theta"], s["g"], s["m"], s["v"], t=s["t"], **adam, **pack)
        return [s[k] for k in ("theta", "m", "v")]
    if rule == "async":
        arn.async_adam_local_step(s["theta"], s["g"], s["m"], s["v"], s["a_g"], s["a_g2"], s["a_s"], t=s["t"], **adam,
                                  **pack)
        return [s[k] for k in ("theta", "m", "v", "a_g", "a_g2", "a_s")]
    arn.async_adam_merge(s["theta_c"], s["m_c"], s["v_c"], s["theta"], s["m"], s["v"], s["a_g"], s["a_g2"], s["a_s"],
                         n_local=5, beta1=0.9, beta2=0.999, **pack)
    return [s[k] for k in ("theta_c", "m_c", "v_c", "theta", "m", "v", "a_g", "a_g2", "a_s")]


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def parameter_count(case):
    inputs, hidden = FC[case["geometry"]]
    return (sum(cout * (cin * k * k + 1) for cin, cout, k, _ in CONVS[case["geometry"]]) + hidden * (inputs + 1) +
            head_rows(case) * (hidden + 1))


def work(case):
    n = parameter_count(case)
    if case["kind"] == "update":
        # the rule's own arrays, and the 16-bit copy of the parameters written by the re-pack
        return dict(bytes=(UPDATE_BYTES[case["rule"]] + 2) * n, flops=12 * n)
    inputs, hidden = FC[case["geometry"]]
    first = 2 * CONVS[case["geometry"]][0][1] * CONVS[case["geometry"]][0][0] * 64 * CONVS[case["geometry"]][0][3]
    forward = sum(2 * cin * cout * k * k * p for cin, cout, k, p in CONVS[case["geometry"]])
    forward += 2 * inputs * hidden + 2 * hidden * head_rows(case)
    batch, frame = case["batch"], 4 * FRAME[case["geometry"]][0] * FRAME[case["geometry"]][1]
    if case["kind"] in ("forward", "act"):
        out = 8 if case["kind"] == "act" else 4 * (head_rows(case) + case["actions"] + 2)
        return dict(bytes=2 * n + batch * (frame + out), flops=batch * forward)
    # forward, weight gradient, and input gradient of every layer but the first; 16-bit weights in, fp32 gradient out
    bootstrapped = case["objective"] in ("c51", "dqn")
    passes = {"c51": 1, "dqn": 2}.get(case["objective"], 0)   # forward passes on the next states
    flops = batch * (3 * forward - first + passes * forward)
    size = 2 * n * (2 if bootstrapped else 1) + 4 * n + batch * (frame * (2 if bootstrapped else 1) + 16)
    if case["kind"] == "learn":
        size, flops = size + (UPDATE_BYTES["rmsprop"] + 2) * n, flops + 6 * n
    return dict(bytes=size, flops=flops)


def tolerance(case):
    if case["kind"] == "update":
        return dict(rel=1e-5)
    # Contractions of 16-bit operands with fp32 sums.  Greedy, drawn and bootstrapped actions are decisions on such
    # values: near ties may fall either way.
    return dict(rel=1e-2, differ=0.01)
