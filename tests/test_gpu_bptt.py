"""GPU parity of the backward pass: marl_qnet_grad through the C ABI against the fp64 oracle, tensor by
tensor of the packed gradient.  Bar: every entry within REL * max |oracle tensor| (plus a small absolute
floor) of the oracle; REL = 1e-3 for fp32 networks (split-bf16 products, fp32 sums over all samples), 3e-2
for bf16 networks (weights, activations and the recurrent adjoints rounded to bf16).  The first layer's
ReLU is a yes/no decision taken on forward values: where the oracle's pre-activation is within the
forward tolerance of zero the two sides may decide differently, so the entries of W1 and b1 get, on top,
the oracle's ambiguity budget for that band (the summed magnitude of exactly those samples' terms)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import bptt_oracle as bpo
from paper_2205_05248_amd import binding, workloads as wl
import parity_util as pu

pytestmark = pytest.mark.gpu
REL = {"fp32": 1e-3, "bf16": 3e-2}
# Half-width of the band of first-layer pre-activations in which the two sides may switch a unit differently:
# the forward error of that pre-activation against fp64.  A bf16 network's kernels round every observation entry
# to bf16 before the first-layer product; the ReLU is a decision, and both sides take a decision on the same
# values: the oracle runs in its bf16-input mode (its own rounding routine, pinned against a library cast).  What
# is left is rounding in the sums.  bf16 networks: products of two bf16 values are exact in fp32, the sum of up
# to 364 of them in fp32 is off by a few 1e-7 at pre-activations of order one.  fp32 networks: each operand is
# split into two bf16 planes and the low-by-low product dropped, 2^-17 of each product, a few 1e-6 over the sum.
RELU_BAND = {"fp32": 2e-5, "bf16": 1e-6}
# The ambiguity budget that band may claim, as a share of the tensor's largest reference value: a band wide
# enough to hide an error in W1 or b1 fails here.
BUDGET_CAP = 0.02


def oracle_grad(cfg, w, u, g, band=None):
    dtype = cfg["dtype"]
    return bpo.qnet_grad(wl.dims(cfg), pu.oracle_weights(cfg, w), u["obs"], u["actions"], u["filled"], g.astype(np.float64),
                         relu_band=RELU_BAND[dtype] if band is None else band, inputs_as_bf16=dtype == "bf16")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


def gpu_grad(net, cfg, u, g, workspace=None):
    d = pu.to_dev(u, ["obs", "actions", "filled"])
    B, T = u["actions"].shape[:2]
    need = net.grad_workspace_bytes(B, T)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if workspace is None else workspace
    ws.fill_(0xFF)                                   # NaN patterns: nothing may be read before it is written
    n_params = wl.param_count(*wl.dims(cfg))
    out = torch.full((n_params,), float("nan"), device="cuda")
    net.grad(d["obs"], d["actions"], d["filled"], torch.from_numpy(g.astype(np.float32)).cuda(), ws, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def compare(cfg, got, want, amb):
    rel = REL[cfg["dtype"]]
    assert np.isfinite(got).all()
    worst, bad = {}, []
    for name, (a, b, _) in wl.weight_slices(*wl.dims(cfg)).items():
        scale = np.abs(want[a:b]).max()
        err = np.abs(got[a:b] - want[a:b])
        worst[name] = err.max() / max(scale, 1e-30)
        if name not in ("W1", "b1"):
            assert amb[a:b].max() == 0
        assert amb[a:b].max() <= BUDGET_CAP * max(scale, 1e-30), (name, amb[a:b].max() / max(scale, 1e-30))
        over = err - (rel * scale + 1e-6 + amb[a:b])
        if over.max() > 0:
            bad.append(f"{name}: max err {err.max():.3e} against scale {scale:.3e}, budget up to {amb[a:b].max():.3e}")
    print(cfg["name"], {k: f"{v:.1e}" for k, v in worst.items()}, "budget/scale W1 %.1e" % (
        amb[:wl.weight_slices(*wl.dims(cfg))["W1"][1]].max() / np.abs(want[:wl.weight_slices(*wl.dims(cfg))["W1"][1]]).max()))
    assert not bad, bad
    return worst


CASES = [(0, 4, 6, {}), (0, 32, 25, {}), (1, 5, 9, {}), (2, 7, 12, {}), (3, 33, 5, {}), (4, 3, 11, {}),
         # the widest first layer and more than sixteen agents with fp32 weights; a bf16 network with H = 64
         (4, 3, 7, dict(H=64, D=150, dtype="fp32")), (1, 6, 8, dict(dtype="bf16")),
         # odd shapes: one agent, odd observation and action counts, the most actions, a hidden-128 network with few inputs
         (0, 5, 13, dict(N=1, D=7, A=5)), (0, 3, 6, dict(N=17, D=33, A=64, dtype="bf16")),
         (4, 4, 9, dict(N=2, D=160, A=4)), (1, 1, 40, dict(N=3, D=1, A=7)),
         # bf16 networks over sixteen slots or more: the slots are walked in two launches (an odd count: halves of
         # eight and nine) and the products run per half; the last one's first layer keeps the narrow loads
         (4, 2, 17, {}), (1, 3, 24, dict(dtype="bf16")), (0, 2, 16, dict(N=17, D=33, A=64, dtype="bf16")),
         # two launches of unequal halves, for 64 hidden units on tiles of eight rows, with odd and even counts on either side;
         # the halves fill more chunks of partial sums together than all slots at once would
         (2, 3, 17, dict(N=5, D=96, dtype="bf16")), (2, 12, 17, dict(N=5, D=96, dtype="bf16")),
         (2, 2, 19, dict(N=5, D=96, dtype="bf16")), (2, 3, 21, dict(N=5, D=96, dtype="bf16")),
         (2, 12, 61, dict(N=5, D=96, dtype="bf16")), (4, 12, 17, dict(N=5, D=96, A=11)),
         # one launch, just past the samples up to which a chunk of a bf16 network has 64
         (2, 37, 14, dict(N=5, D=55, dtype="bf16")),
         # more tiles of sixteen rows than compute units: two workgroups of a bf16 network share one, fp32 ones follow one another
         (2, 823, 5, dict(N=5, D=24, dtype="bf16")), (2, 823, 3, dict(N=5, D=24))]


@pytest.mark.parametrize("ci,B,T,over", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_gradient_matches_the_oracle(ci, B, T, over):
    cfg = dict(wl.config(ci), B=B, T=T, **over)
    dims = wl.dims(cfg)
    w = wl.make_weights(cfg, 0)
    net = binding.QNet(dims, w, cfg["dtype"])
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    g = np.random.default_rng(ci).normal(size=(B, T, dims[0])).astype(np.float32)
    got = gpu_grad(net, cfg, u, g)
    want, amb = oracle_grad(cfg, w, u, g)
    compare(cfg, got, want, amb)
    # the same call again: identical bits (fixed summation order)
    again = gpu_grad(net, cfg, u, g)
    np.testing.assert_array_equal(again, got)
    net.close()


# The reverse recurrence of a 64-unit network with few rows (tiles of eight) walks the slots two a round, an odd one first, with the
# inputs of the slots before in flight: the fewest slots, odd and even, and row counts on both sides of a tile.
@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("dtype,B,N", [("fp32", 1, 2), ("fp32", 17, 1), ("bf16", 5, 3), ("bf16", 16, 1)])
def test_gradient_of_the_fewest_slots(dtype, B, N, T):
    cfg = dict(wl.config(0), dtype=dtype, N=N, B=B, T=T)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    g = np.random.default_rng(7).standard_normal(u["actions"].shape).astype(np.float32)
    net = binding.QNet(wl.dims(cfg), w, dtype)
    compare(cfg, gpu_grad(net, cfg, u, g), *oracle_grad(cfg, w, u, g))
    net.close()


# With more rows than tiles of eight are taken for, a 64-unit network walks the slots on tiles of sixteen, in an unrolled loop of
# three with two slots of inputs in flight: the fewest slots and every remainder in one launch, and, for a bf16 network, every
# remainder of either half of two launches, whose second goes on from what the first carried.
@pytest.mark.parametrize("dtype,B,T,N", [(d, 683, T, 3) for d in ("fp32", "bf16") for T in (1, 2, 3, 4)]
                         + [("bf16", 257, 17, 5), ("bf16", 257, 19, 5), ("bf16", 257, 21, 5), ("bf16", 1024, 18, 3)])
def test_gradient_on_tiles_of_sixteen_rows(dtype, B, T, N):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    eights, two_launches = -(-B * N // 8), dtype == "bf16" and T >= 16 and 2 * -(-B * N // 16) <= 3 * n_cu // 2
    assert eights > (5 * n_cu // 8 if two_launches else n_cu) and two_launches == (T >= 16)
    cfg = dict(wl.config(0), dtype=dtype, N=N, D=8, A=5, B=B, T=T)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    # one sign: the sums grow with the samples as the oracle's ambiguity budget does
    g = np.abs(np.random.default_rng([B, T, N]).normal(size=(B, T, N))).astype(np.float32)
    net = binding.QNet(wl.dims(cfg), w, dtype)
    got = gpu_grad(net, cfg, u, g)
    compare(cfg, got, *oracle_grad(cfg, w, u, g))
    assert (gpu_grad(net, cfg, u, g) == got).all()
    net.close()


def test_full_size_launch_on_a_few_live_episodes():
    """The workload's full batch in the launch configuration the benchmark times; the upstream gradient is
    non-zero for three episodes only, so the oracle has to walk just those (the sum is linear in it), while
    every tile, chunk and reduction of the full-size launch takes part."""
    cfg = wl.config(4)
    dims = wl.dims(cfg)
    B, T = cfg["B"], cfg["T"]
    w = wl.make_weights(cfg, 0)
    net = binding.QNet(dims, w, cfg["dtype"])
    u = wl.make_unroll_inputs(cfg)
    live = [0, 37, B - 1]
    g = np.zeros((B, T, dims[0]), np.float32)
    g[live] = np.random.default_rng(5).normal(size=(len(live), T, dims[0])).astype(np.float32)
    got = gpu_grad(net, cfg, u, g)
    sub = {k: np.ascontiguousarray(u[k][live]) for k in ("obs", "actions", "filled")}
    want, amb = oracle_grad(cfg, w, sub, g[live])
    compare(cfg, got, want, amb)
    net.close()


def test_edge_shapes_and_argument_errors():
    cfg = dict(wl.config(1), B=1, T=1)
    dims = wl.dims(cfg)
    w = wl.make_weights(cfg, 0)
    net = binding.QNet(dims, w, cfg["dtype"])
    # one episode of one step, unfilled steps, and an all-zero upstream gradient
    u = wl.make_unroll_inputs(cfg, B=1, T=1)
    u["filled"][:] = 1
    g = np.ones((1, 1, dims[0]), np.float32)
    want, amb = oracle_grad(cfg, w, u, g)
    compare(cfg, gpu_grad(net, cfg, u, g), want, amb)
    u["filled"][:] = 0
    assert np.abs(gpu_grad(net, cfg, u, g)).max() == 0
    u2 = wl.make_unroll_inputs(cfg, B=3, T=4)
    assert np.abs(gpu_grad(net, cfg, u2, np.zeros((3, 4, dims[0]), np.float32))).max() == 0
    # arguments
    lib, vp = binding.load(), ctypes.c_void_p
    need = ctypes.c_size_t(0)
    assert lib.marl_qnet_grad_workspace_bytes(vp(net.handle), 3, 4, ctypes.byref(need)) == 0 and need.value > 0
    assert lib.marl_qnet_grad_workspace_bytes(vp(net.handle), 0, 4, ctypes.byref(need)) == -2
    assert lib.marl_qnet_grad_workspace_bytes(vp(net.handle), 3, 0, ctypes.byref(need)) == -2
    assert lib.marl_qnet_grad_workspace_bytes(None, 3, 4, ctypes.byref(need)) == -1
    d = pu.to_dev(u2, ["obs", "actions", "filled"])
    gq = torch.zeros(3, 4, dims[0], device="cuda")
    bytes_needed = net.grad_workspace_bytes(3, 4)
    ws = torch.empty(bytes_needed + 256, dtype=torch.uint8, device="cuda")
    out = torch.zeros(wl.param_count(*dims), device="cuda")
    call = lambda ws_ptr, ws_bytes, out_ptr: lib.marl_qnet_grad(
        vp(net.handle), 3, 4, vp(d["obs"].data_ptr()), vp(d["actions"].data_ptr()), vp(d["filled"].data_ptr()),
        vp(gq.data_ptr()), ws_ptr, ws_bytes, out_ptr, None)
    assert call(vp(ws.data_ptr()), bytes_needed - 1, vp(out.data_ptr())) == -2        # workspace too small
    assert call(vp(ws.data_ptr() + 4), bytes_needed, vp(out.data_ptr())) == -5        # misaligned
    assert call(None, bytes_needed, vp(out.data_ptr())) == -1
    assert call(vp(ws.data_ptr()), bytes_needed, None) == -1
    assert call(vp(ws.data_ptr()), bytes_needed, vp(out.data_ptr())) == 0
    torch.cuda.synchronize()
    net.close()
    # a network the fused kernels do not hold is refused, not served some other way
    big = dict(wl.config(4), dtype="fp32")
    net = binding.QNet(wl.dims(big), wl.make_weights(big, 0), "fp32")
    assert lib.marl_qnet_grad_workspace_bytes(vp(net.handle), 3, 4, ctypes.byref(need)) == -2
    net.close()


@pytest.mark.parametrize("ci,B,T,two", [(0, 5, 9, True), (1, 6, 8, False), (4, 3, 11, True)])
def test_unroll_that_keeps_activations_feeds_the_backward_pass(ci, B, T, two):
    """marl_unroll_td_keep returns what marl_unroll_td returns and leaves the activations; marl_qnet_grad_kept on
    them returns what marl_qnet_grad returns.  Both bit for bit."""
    cfg = dict(wl.config(ci), B=B, T=T)
    dims = wl.dims(cfg)
    N, D, A, H = dims
    net = binding.QNet(dims, wl.make_weights(cfg, 0), cfg["dtype"])
    target = binding.QNet(dims, wl.make_weights(cfg, 1), cfg["dtype"]) if two else None
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    d = pu.to_dev(u, ["obs", "avail", "actions", "reward", "terminated", "filled"])
    g = torch.from_numpy(np.random.default_rng(ci).normal(size=(B, T, N)).astype(np.float32)).cuda()
    ws = torch.empty(net.grad_workspace_bytes(B, T), dtype=torch.uint8, device="cuda")
    n_params = wl.param_count(*dims)
    plain = pu.gpu_unroll(net, target, cfg, u)
    ws.fill_(0xFF)
    ref = torch.full((n_params,), float("nan"), device="cuda")
    net.grad(d["obs"], d["actions"], d["filled"], g, ws, ref)
    torch.cuda.synchronize()
    ws.fill_(0xFF)
    outs = [torch.full((B, T, N), float("nan"), device="cuda") for _ in range(3)]
    q_all = torch.full((B, T + 1, N, A), float("nan"), device="cuda")
    net.unroll_td_keep(target, d["obs"], d["avail"], d["actions"], d["reward"], d["terminated"], d["filled"], u["gamma"],
                       *outs, ws, q_all)
    got = torch.full((n_params,), float("nan"), device="cuda")
    net.grad(d["obs"], d["actions"], d["filled"], g, ws, got, kept=True)
    torch.cuda.synchronize()
    for o, k in zip(outs + [q_all], ("q_taken", "next_max", "td_target", "q_all")):
        np.testing.assert_array_equal(o.cpu().numpy(), plain[k])
    assert torch.equal(got, ref)
    lib, vp = binding.load(), ctypes.c_void_p
    args = (vp(net.handle), vp(net.handle), B, T, vp(d["obs"].data_ptr()), vp(d["avail"].data_ptr()), vp(d["actions"].data_ptr()),
            vp(d["reward"].data_ptr()), vp(d["terminated"].data_ptr()), vp(d["filled"].data_ptr()), 0.9,
            vp(outs[0].data_ptr()), vp(outs[1].data_ptr()), vp(outs[2].data_ptr()), None)
    assert lib.marl_unroll_td_keep(*args, vp(ws.data_ptr()), ws.numel() - 1, None) == -2
    assert lib.marl_unroll_td_keep(*args, None, ws.numel(), None) == -1
    net.set_kernels(binding.KERNELS_TILE32)
    assert lib.marl_unroll_td_keep(*args, vp(ws.data_ptr()), ws.numel(), None) == -2          # the two-kernel family keeps nothing
    net.close()
    if target is not None:
        target.close()
