"""The work a user of this framework has it do, as cases to be timed: sizes, inputs, one pass, what the pass
cannot do without, and how closely two correct implementations agree.

Kinds of case
  decide         a worker's decision step for all its environments (QNet.act_step)
  decide_listed  the same for the environments that have delivered an observation (QNet.act_step_indexed)
  unroll         the learner's forward half: TD targets over a batch of episodes (QNet.unroll_td)
  unroll_pool    double-estimator targets, the batch read in place from a replay pool (QNet.unroll_td_double)
  learn          a whole learner iteration: unroll that keeps its activations, mixing network forward and
                 backward, back-propagation through time, both RMSprop updates
Sizes of the listed cases are those of workloads.CONFIGS (the paper's scenarios and the scale-up) or odd ones
between them; draw() spreads over the whole range.
"""
import math

import numpy as np
import torch

from paper_2205_05248_amd import binding, workloads as wl

GAMMA = 0.99
RMS_ALPHA, RMS_EPS = 0.99, 1e-5
# Late in a learning-rate schedule: repeated passes over one batch stay at the same point of the training.
LEARN_RATE = 1e-6


def listed():
    cases = [
        # The smallest call: a worker with eight environments of the 3m scenario; the Q values stay inside.
        dict(name="decide_tiny", kind="decide", E=8, N=3, D=30, A=9, H=64, dtype="fp32", want_q=False),
        # A large worker on a small scenario (5m_vs_6m), fp32, observation size not a multiple of four.
        dict(name="decide_5m_vs_6m", kind="decide", E=4096, N=5, D=55, A=12, H=64, dtype="fp32", want_q=False),
        # The scale-up worker: 32 agents, hidden 128, bf16 weights, Q values wanted.
        dict(name="decide_scaleup", kind="decide", E=2048, N=32, D=300, A=40, H=128, dtype="bf16", want_q=True),
        # Asynchronous actors: a ragged part of a worker's environments, odd sizes throughout.
        dict(name="decide_listed", kind="decide_listed", E=1000, listed=357, N=7, D=93, A=13, H=128, dtype="bf16", want_q=False),
        # Evaluation of a learner batch of the 8m scenario without an update (fp32, every slot's Q values kept).
        dict(name="unroll_8m", kind="unroll", B=32, T=120, N=8, D=80, A=14, H=64, dtype="fp32", want_q=True),
        # The scale-up batch, forward half alone.
        dict(name="unroll_scaleup", kind="unroll", B=64, T=200, N=32, D=300, A=40, H=128, dtype="bf16", want_q=False),
        # Double-estimator targets of a batch sampled from a replay pool; the larger hidden layer in fp32.
        dict(name="unroll_pool_h128", kind="unroll_pool", pool=200, B=61, T=70, N=5, D=55, A=12, H=128, dtype="fp32", want_q=False),
        # The smallest learner iteration (3m): every launch is short and their number counts.
        dict(name="learn_3m", kind="learn", B=4, T=60, N=3, D=30, A=9, H=64, S=48, M=32, dtype="fp32"),
        # An ordinary learner iteration (2s3z).
        dict(name="learn_2s3z", kind="learn", B=64, T=120, N=5, D=96, A=11, H=64, S=120, M=32, dtype="fp32"),
        # Odd sizes, bf16 weights on the smaller hidden layer.
        dict(name="learn_ragged", kind="learn", B=37, T=83, N=5, D=55, A=12, H=64, S=98, M=32, dtype="bf16"),
        # The largest: the scale-up learner iteration.
        dict(name="learn_scaleup", kind="learn", B=64, T=200, N=32, D=300, A=40, H=128, S=512, M=32, dtype="bf16"),
    ]
    return cases


def _log_int(rng, low, high):
    return max(low, min(high, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def draw(rng):
    kind = rng.choice(["decide", "decide_listed", "unroll", "unroll_pool", "learn", "learn"])
    H, dtype = rng.choice([(64, "fp32"), (64, "bf16"), (128, "bf16"), (128, "fp32")])
    if kind == "learn" and (H, dtype) == (128, "fp32"):           # the backward pass does not serve this pair
        H = 64
    N = _log_int(rng, 2, 32)
    widest = 160 if kind == "learn" and dtype == "fp32" else 300
    D = _log_int(rng, 20, widest)
    A = rng.randint(5, 40)
    case = dict(kind=kind, N=N, D=D, A=A, H=H, dtype=dtype)
    if kind in ("decide", "decide_listed"):
        case.update(E=_log_int(rng, 1, min(8192, 65536 // N)), want_q=rng.random() < 0.5)
        if kind == "decide_listed":
            case["listed"] = rng.randint(1, case["E"])
        return case
    T = rng.randint(25, 200)
    most = 409600 if dtype == "bf16" else 102400                  # agent steps of a batch (fp32 arithmetic costs about three times as much)
    B = _log_int(rng, 4, max(4, min(128, most // (T * N))))
    case.update(B=B, T=T)
    if kind == "learn":
        case.update(S=_log_int(rng, 32, 512), M=rng.choice([16, 32, 32, 64]))
        return case
    case["want_q"] = rng.random() < 0.5
    if kind == "unroll_pool":
        case["pool"] = rng.randint(B, 2 * B)
    return case


# ------------------------------------------------------------------------------------------ inputs
class _Draws:
    """Random device tensors of one seed."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.gen, device="cuda")

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda")

    def observations(self, *shape):
        """Values in [0, 1), about a third of them zero (units out of sight)."""
        return self.uniform(*shape) * (self.uniform(*shape) >= 0.3)

    def available(self, *shape):
        """Each action available with probability 0.7, action 0 always."""
        avail = (self.uniform(*shape) < 0.7).to(torch.uint8)
        avail[..., 0] = 1
        return avail


def _nets(case, seed, count):
    dims = (case["N"], case["D"], case["A"], case["H"])
    weights = [wl.make_weights(dict(case, seed=int(seed) & 0x7FFFFFFF), stream) for stream in range(count)]
    return [binding.QNet(dims, w, case["dtype"]) for w in weights], weights


def _episodes(draws, case, count):
    """`count` episodes of up to T steps, padded with zeros after their end, actions uniform over the available."""
    T, N, D, A = case["T"], case["N"], case["D"], case["A"]
    length = torch.randint(T // 2, T + 1, (count, 1), generator=draws.gen, device="cuda")
    inside = torch.arange(T + 1, device="cuda")[None, :] <= length
    step = torch.arange(T, device="cuda")[None, :]
    obs = draws.observations(count, T + 1, N, D) * inside[:, :, None, None]
    avail = draws.available(count, T + 1, N, A) * inside[:, :, None, None]
    avail[..., 0] = 1
    score = draws.uniform(count, T, N, A) * avail[:, :T]
    filled = (step < length).to(torch.uint8)
    return dict(obs=obs, avail=avail, actions=score.argmax(-1).to(torch.int32), inside=inside,
                reward=draws.normal(count, T) * filled, filled=filled,
                terminated=((step == length - 1) & (length < T)).to(torch.uint8))


def prepare(case, seed):
    draws = _Draws(seed)
    kind, N, D, A, H = case["kind"], case["N"], case["D"], case["A"], case["H"]
    state = dict(case=case)
    if kind in ("decide", "decide_listed"):
        E = case["E"]
        (state["net"],), _ = _nets(case, seed, 1)
        state.update(
            obs=draws.observations(E, N, D), avail=draws.available(E, N, A), h_in=draws.uniform(E, N, H) * 2 - 1,
            reset=(draws.uniform(E) < 0.02).to(torch.uint8),
            step_t=torch.randint(0, 120, (E,), generator=draws.gen, device="cuda", dtype=torch.int32),
            seed=int(seed), h_out=torch.zeros(E, N, H, device="cuda"),
            action=torch.zeros(E, N, dtype=torch.int32, device="cuda"),
            q=torch.zeros(E, N, A, device="cuda") if case["want_q"] else None)
        if kind == "decide_listed":
            state["index"] = torch.randperm(E, generator=draws.gen, device="cuda")[: case["listed"]].to(torch.int32).contiguous()
        return state
    B, T = case["B"], case["T"]
    (online, target), weights = _nets(case, seed, 2)
    state.update(online=online, target=target, **_episodes(draws, case, case.get("pool", B)))
    for name in ("q_taken", "next_max", "td_target"):
        state[name] = torch.zeros(B, T, N, device="cuda")
    if kind != "learn":
        state["q_all"] = torch.zeros(B, T + 1, N, A, device="cuda") if case["want_q"] else None
        binding.marl_qnet_reserve_unroll(online.handle, B, T)
        if kind == "unroll_pool":
            binding.marl_qnet_reserve_unroll(target.handle, B, T)
            state["next_action"] = torch.zeros(B, T, N, dtype=torch.int32, device="cuda")
            state["index"] = torch.randint(0, case["pool"], (B,), generator=draws.gen, device="cuda", dtype=torch.int32)
        return state
    S, M = case["S"], case["M"]
    mcfg = dict(seed=int(seed) & 0x7FFFFFFF, N=N, S=S)
    mdims = (N, M, S)
    mweights = [_mixer_weights(mcfg, mdims, stream) for stream in range(2)]
    mixer, mixer_target = (binding.Mixer(mdims, w, case["dtype"]) for w in mweights)
    state.update(
        mixer=mixer, mixer_target=mixer_target,
        state=draws.observations(B, T + 1, S) * state["inside"][:, :, None],
        zero=torch.zeros(B, T, device="cuda"), loss=torch.zeros(2, device="cuda"), grad_q=torch.zeros(B, T, N, device="cuda"),
        work=torch.zeros(online.grad_workspace_bytes(B, T), dtype=torch.uint8, device="cuda"),
        mixer_work=torch.zeros(mixer.grad_workspace_bytes(B, T), dtype=torch.uint8, device="cuda"))
    for name in ("q_total", "y_total", "td_err", "grad_q_total"):
        state[name] = torch.zeros(B, T, device="cuda")
    for name, w in (("", weights[0]), ("mixer_", mweights[0])):
        state[name + "weights"] = torch.from_numpy(w.copy()).cuda()
        state[name + "grad"] = torch.zeros(w.size, device="cuda")
        state[name + "sq_avg"] = draws.uniform(w.size) * 1e-3
    return state


def _mixer_weights(cfg, mdims, stream):
    """As workloads.make_mixer_weights, for any number of hidden units of the mixer."""
    rng = np.random.default_rng([cfg["seed"], 4000 + stream])
    parts = {}
    for name, (_, _, shape) in wl.mixer_slices(*mdims).items():
        bound = 1.0 / np.sqrt(shape[-1]) if len(shape) == 2 or name == "v2" else 0.05
        parts[name] = rng.uniform(-bound, bound, shape)
    return wl.pack_mixer(mdims, parts)


# ------------------------------------------------------------------------------------------ one pass
def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind in ("decide", "decide_listed"):
        epsilon = 0.05
        if kind == "decide":
            s["net"].act_step(s["obs"], s["avail"], s["h_in"], s["reset"], s["step_t"], epsilon, s["seed"],
                              s["h_out"], s["action"], s["q"])
        else:
            s["net"].act_step_indexed(s["index"], s["obs"], s["avail"], s["h_in"], s["reset"], s["step_t"], epsilon, s["seed"],
                                      s["h_out"], s["action"], s["q"])
        return {k: s[k] for k in ("h_out", "action", "q") if s[k] is not None}
    batch = [s[k] for k in ("obs", "avail", "actions", "reward", "terminated", "filled")]
    outputs = [s[k] for k in ("q_taken", "next_max", "td_target")]
    named = ["q_taken", "next_max", "td_target"]
    if kind == "unroll":
        s["online"].unroll_td(s["target"], *batch, GAMMA, *outputs, s["q_all"])
        named += ["q_all"]
    elif kind == "unroll_pool":
        s["online"].unroll_td_double(s["target"], *batch, GAMMA, *outputs, s["next_action"], s["q_all"], s["index"])
        named += ["q_all", "next_action"]
    else:
        s["online"].unroll_td_keep(s["target"], *batch, GAMMA, *outputs, s["work"])
        s["mixer"].td(s["mixer_target"], s["state"], s["q_taken"], s["next_max"], s["reward"], s["terminated"], s["filled"], GAMMA,
                      s["q_total"], s["y_total"], s["td_err"], s["loss"])
        # dL/dQ_total = -2 td_err / number of transitions, in one element-wise kernel
        torch.addcdiv(s["zero"], s["td_err"], s["loss"][1], value=-2.0, out=s["grad_q_total"])
        s["mixer"].grad(s["state"], s["q_taken"], s["grad_q_total"], s["mixer_work"], s["grad_q"], s["mixer_grad"])
        s["online"].grad(s["obs"], s["actions"], s["filled"], s["grad_q"], s["work"], s["grad"], kept=True)
        s["online"].rmsprop_step(s["weights"], s["grad"], s["sq_avg"], LEARN_RATE, RMS_ALPHA, RMS_EPS)
        s["mixer"].rmsprop_step(s["mixer_weights"], s["mixer_grad"], s["mixer_sq_avg"], LEARN_RATE, RMS_ALPHA, RMS_EPS)
        named += ["q_total", "y_total", "td_err", "loss", "grad_q", "grad", "mixer_grad", "weights", "mixer_weights",
                  "sq_avg", "mixer_sq_avg"]
    return {k: s[k] for k in named if s[k] is not None}


# ------------------------------------------------------------------------------------------ the same in 64 bits
def _held(parts, dtype):
    """float64 tensors of a parameter set as a handle of this type holds it: matrices of a bf16 one rounded once."""
    tensors = {k: torch.as_tensor(v).cuda() for k, v in parts.items()}
    if dtype == "bf16":
        tensors = {k: v.bfloat16().float() if v.dim() == 2 else v for k, v in tensors.items()}
    return {k: v.double() for k, v in tensors.items()}


def _gru_step(w, x, h):
    H = h.shape[-1]
    gx, gh = x @ w["W_ih"].T + w["b_ih"], h @ w["W_hh"].T + w["b_hh"]
    r, z = torch.sigmoid(gx[..., :2 * H] + gh[..., :2 * H]).split(H, -1)
    n = torch.tanh(gx[..., 2 * H:] + r * gh[..., 2 * H:])
    return (1 - z) * n + z * h


def _first_layer(w, obs):
    D = obs.shape[-1]
    return torch.relu(obs @ w["W1"][:, :D].T + w["W1"][:, D:].T + w["b1"])          # the agent's id is a one-hot: a column


def _q_values(w, obs):
    """Q [B, slots, N, A] of whole episodes, hidden state zero before the first slot."""
    x = _first_layer(w, obs)
    h, hidden = torch.zeros_like(x[:, 0]), []
    for s in range(x.shape[1]):
        h = _gru_step(w, x[:, s], h)
        hidden.append(h)
    return torch.stack(hidden, 1) @ w["W2"].T + w["b2"]


def _mixed(w, q, state):
    """Q_total [B, T] of agents' values q [B, T, N] under global states [B, T, S]."""
    M = w["v2"].numel()
    w1 = (state @ w["Hw1"].T + w["hb1"]).abs().unflatten(-1, (-1, M))
    hidden = torch.nn.functional.elu((q[..., None] * w1).sum(-2) + state @ w["Hb1"].T + w["hbb1"])
    offset = torch.relu(state @ w["V1"].T + w["c1"]) @ w["v2"] + w["c2"]
    return (hidden * (state @ w["Hw2"].T + w["hb2"]).abs()).sum(-1) + offset


def _packed(grads, like):
    return torch.cat([grads[k].reshape(-1) for k in like])


def _rmsprop(weights, grad, sq_avg):
    sq_avg = RMS_ALPHA * sq_avg.double() + (1 - RMS_ALPHA) * grad ** 2
    return weights.double() - LEARN_RATE * grad / (sq_avg.sqrt() + RMS_EPS), sq_avg


def exact(case, seed):
    """What run() returns, as plain float64 tensor operations give it for the networks that the handles hold. Actions
    are left out (they depend on the library's random numbers), and with the double estimator whatever hangs on its
    choice of action (two that tie within rounding may be taken either way)."""
    s = prepare(case, seed)
    kind, dims = case["kind"], wl.dims(case)
    nets = [_held(wl.unpack_weights(dims, wl.make_weights(dict(case, seed=int(seed) & 0x7FFFFFFF), stream)), case["dtype"])
            for stream in range(2)]
    if kind in ("decide", "decide_listed"):
        envs = s["index"].long() if kind == "decide_listed" else slice(None)
        w = nets[0]
        h = s["h_in"][envs].double() * (1 - s["reset"][envs].double())[:, None, None]
        h_new = _gru_step(w, _first_layer(w, s["obs"][envs].double()), h)
        out = dict(h_out=s["h_out"].double(), action=None)
        out["h_out"][envs] = h_new
        if s["q"] is not None:
            out["q"] = s["q"].double()
            out["q"][envs] = h_new @ w["W2"].T + w["b2"]
        return out
    batch = {k: s[k] for k in ("obs", "avail", "actions", "reward", "terminated", "filled")}
    if kind == "unroll_pool":
        batch = {k: v[s["index"].long()] for k, v in batch.items()}
    obs, filled, running = batch["obs"].double(), batch["filled"].double(), 1 - batch["terminated"].double()
    leaves = {k: v.requires_grad_(kind == "learn") for k, v in nets[0].items()}
    q_all = _q_values(leaves, obs)
    q_taken = q_all[:, :-1].gather(-1, batch["actions"].long()[..., None])[..., 0] * filled[..., None]
    with torch.no_grad():
        q_target = _q_values(nets[1], obs)[:, 1:].masked_fill(batch["avail"][:, 1:] == 0, -math.inf)
        next_max = q_target.max(-1).values * filled[..., None]
        td_target = (batch["reward"].double()[..., None] + GAMMA * running[..., None] * next_max) * filled[..., None]
    out = dict(q_taken=q_taken, next_max=next_max, td_target=td_target)
    if kind != "learn":
        if s["q_all"] is not None:
            out["q_all"] = q_all
        if kind == "unroll_pool":
            out.update(next_max=None, td_target=None, next_action=None)
        return out
    mdims = (case["N"], case["M"], case["S"])
    mixers = []
    for stream in range(2):
        packed = _mixer_weights(dict(seed=int(seed) & 0x7FFFFFFF, N=case["N"], S=case["S"]), mdims, stream)
        mixers.append(_held({k: packed[a:b].reshape(shape) for k, (a, b, shape) in wl.mixer_slices(*mdims).items()}, case["dtype"]))
    mleaves = {k: v.requires_grad_() for k, v in mixers[0].items()}
    states = s["state"].double()
    q_total = _mixed(mleaves, q_taken, states[:, :-1])
    with torch.no_grad():
        y_total = batch["reward"].double() + GAMMA * running * _mixed(mixers[1], next_max, states[:, 1:])
        td_err = (y_total - q_total) * filled
        loss = torch.stack([(td_err ** 2).sum(), filled.sum()])
    names = list(leaves.values()) + list(mleaves.values()) + [q_taken]
    grads = torch.autograd.grad(q_total, names, -2.0 * td_err / loss[1])
    grad = _packed(dict(zip(leaves, grads)), leaves)
    mixer_grad = _packed(dict(zip(mleaves, grads[len(leaves):])), mleaves)
    weights, sq_avg = _rmsprop(s["weights"], grad, s["sq_avg"])
    mixer_weights, mixer_sq_avg = _rmsprop(s["mixer_weights"], mixer_grad, s["mixer_sq_avg"])
    out.update(q_total=q_total, y_total=y_total, td_err=td_err, loss=loss, grad_q=grads[-1], grad=grad, mixer_grad=mixer_grad,
               weights=weights, mixer_weights=mixer_weights, sq_avg=sq_avg, mixer_sq_avg=mixer_sq_avg)
    return {k: v.detach() for k, v in out.items()}


# ------------------------------------------------------------------------------------------ accounting
def work(case):
    kind, N, D, A, H = case["kind"], case["N"], case["D"], case["A"], case["H"]
    weight = 4 if case["dtype"] == "fp32" else 2
    params = wl.param_count(N, D, A, H)
    forward = 2 * D * H + 12 * H * H + 2 * H * A                     # of one agent step
    if kind in ("decide", "decide_listed"):
        envs = case["listed"] if kind == "decide_listed" else case["E"]
        rows = envs * N
        per_row = 4 * D + A + 8 * H + 4 + (4 * A if case["want_q"] else 0)
        return {"bytes": rows * per_row + envs * (9 if kind == "decide_listed" else 5) + params * weight, "flops": rows * forward}
    B, T = case["B"], case["T"]
    slots, steps = B * (T + 1) * N, B * T * N
    flops = 2 * slots * forward
    nbytes = slots * (4 * D + A) + steps * (4 + 12) + B * T * 6 + 2 * params * weight
    if kind != "learn":
        nbytes += (4 * slots * A if case["want_q"] else 0) + (4 * steps if kind == "unroll_pool" else 0)
        return {"bytes": nbytes, "flops": flops}
    S, M = case["S"], case["M"]
    mixer_params = wl.mixer_param_count(N, M, S)
    generated = 2 * (N + 3) * M * S                                  # the mixer's state products, per transition
    # backward: both GRU products for the data, both for the weights, fc1's and fc2's weights (one action per sample)
    flops += steps * (24 * H * H + 2 * D * H + 4 * H) + 3 * B * T * generated
    # states, values per transition, dL/dq; weights, their gradients and running squares read and written
    nbytes += 4 * B * (T + 1) * S + 16 * B * T + 4 * steps + 24 * (params + mixer_params)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what was measured: the learner iteration against the same computation with float64
    activations and autograd (fp32 networks: gradients 4e-5 in norm, 1.1e-3 at worst; bf16 networks, whose
    activations are rounded for every product: 2.6e-3 in norm, 1.3e-2 and for gradients 3.2e-2 at worst), the decision
    step and the unrolls against the other kernel family as well (fp32 2e-6 / 2e-5)."""
    fp32, kind = case["dtype"] == "fp32", case["kind"]
    if kind == "unroll_pool":
        # Where two actions tie within rounding the online network's choice may be the other one, and the target
        # network values the two differently: a value in a few thousand (a few hundred in bf16) differs outright.
        return {"rel": 5e-3, "differ": 1e-3} if fp32 else {"rel": 3e-2, "differ": 1e-2}
    if kind == "learn":
        return {"rel": 1.5e-4, "max": 4e-3} if fp32 else {"rel": 1e-2, "max": 1.2e-1}
    return {"rel": 3e-5, "max": 2e-4, "differ": 1e-3} if fp32 else {"rel": 1e-2, "max": 5e-2, "differ": 1e-2}
