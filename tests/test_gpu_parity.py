"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle, element by
element on the same seeded inputs.  Tolerances: max abs error 1e-4 with fp32 weights, 2e-2
with bf16 weights (fp32 accumulation); integer outputs exact outside near-ties."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import marl_oracle as orc
from paper_2205_05248_amd import binding, workloads as wl
import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()                      # a missing library is an error, not a skip
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


def make_net(cfg, stream=0, weights=None, kernels=None):
    w = wl.make_weights(cfg, stream) if weights is None else weights
    net = binding.QNet(wl.dims(cfg), w, cfg["dtype"])
    if kernels is not None:
        net.set_kernels(kernels)
    return net, pu.oracle_weights(cfg, w)


def oracle_act(cfg, w, inp):
    return orc.act_step(wl.dims(cfg), w, inp["obs"], inp["avail"], inp["h_in"], inp["reset"], inp["step_t"],
                        inp["epsilon"], inp["seed"])


def oracle_unroll(cfg, w_on, w_tg, u, rows=None):
    return orc.unroll_td(wl.dims(cfg), w_on, w_tg, u["obs"], u["avail"], u["actions"], u["reward"],
                         u["terminated"], u["filled"], u["gamma"], rows=rows)


# Both kernel families are held to the same bar.
PATHS = [binding.KERNELS_TILE32, binding.KERNELS_FUSED16]
PATH_IDS = ["tile32", "fused16"]
# the decision step has a third implementation (the default where it fits)
ACT_PATHS = PATHS + [binding.KERNELS_STREAM16]
ACT_PATH_IDS = PATH_IDS + ["stream16"]


# ------------------------------------------------------------------ act-step
@pytest.mark.parametrize("path", ACT_PATHS, ids=ACT_PATH_IDS)
@pytest.mark.parametrize("ci", [0, 1, 2, 3, 4])
def test_act_step_full_config(ci, path):
    cfg = wl.config(ci)
    tol = pu.TOL[cfg["dtype"]]
    net, w = make_net(cfg, kernels=path)
    inp = wl.make_act_inputs(cfg)
    ref = oracle_act(cfg, w, inp)
    got = pu.gpu_act(net, cfg, inp)
    ties = pu.compare_act(cfg, inp, got, ref, tol)
    print(f"cfg{ci}: rows={cfg['E'] * cfg['N']} maxerr_q={np.abs(got['q'] - ref['q']).max():.3e} near_ties={ties}")
    differ = int((got["action"] != ref["action"]).sum())
    print(f"cfg{ci}: actions differing from the oracle inside near-ties: {differ}")
    # same call without the optional Q output and with h_out aliasing h_in
    got2 = pu.gpu_act(net, cfg, inp, want_q=False, alias_h=True)
    np.testing.assert_array_equal(got2["action"], got["action"])
    np.testing.assert_array_equal(got2["h_out"], got["h_out"])
    net.close()


@pytest.mark.parametrize("path", ACT_PATHS, ids=ACT_PATH_IDS)
@pytest.mark.parametrize("ci,E", [(0, 1), (0, 5), (0, 11), (1, 3), (1, 37), (3, 13), (3, 203), (3, 1000), (4, 1), (4, 9)])
def test_act_step_ragged_sizes(ci, E, path):
    cfg = wl.config(ci)
    net, w = make_net(cfg, kernels=path)
    for eps in (0.0, 0.5, 1.0):
        inp = wl.make_act_inputs(cfg, E=E, stream=E)
        inp["epsilon"] = eps
        ref = oracle_act(cfg, w, inp)
        got = pu.gpu_act(net, cfg, inp)
        pu.compare_act(cfg, inp, got, ref, pu.TOL[cfg["dtype"]])
        chosen = np.take_along_axis(inp["avail"], got["action"][..., None].astype(np.int64), -1)
        assert chosen.all()
    inp["reset"] = None                                   # optional pointer
    ref = oracle_act(cfg, w, inp)
    got = pu.gpu_act(net, cfg, inp)
    pu.compare_act(cfg, inp, got, ref, pu.TOL[cfg["dtype"]])
    net.close()


def test_act_step_closed_forms_on_gpu():
    cfg = wl.config(0)
    dims = wl.dims(cfg)
    N, D, A, H = dims
    zero = {k: np.zeros(shp) for k, (_, _, shp) in wl.weight_slices(*dims).items()}
    inp = wl.make_act_inputs(cfg, E=21)
    inp["reset"][:] = 0
    # every GRU weight zero: r = z = 1/2, candidate 0 -> h' = h / 2 ; Q = b2
    parts = dict(zero)
    parts["b2"] = np.linspace(-1, 1, A)
    net, _ = make_net(cfg, weights=wl.pack_weights(dims, parts))
    got = pu.gpu_act(net, cfg, inp)
    np.testing.assert_allclose(got["h_out"], inp["h_in"] * 0.5, atol=1e-6)
    np.testing.assert_allclose(got["q"], np.broadcast_to(parts["b2"].astype(np.float32), got["q"].shape), atol=1e-6)
    net.close()
    # update gate saturated: h' = h
    parts = {k: np.array(v) for k, v in wl.unpack_weights(dims, wl.make_weights(cfg)).items()}
    parts["b_ih"][H:2 * H] = 40.0
    net, _ = make_net(cfg, weights=wl.pack_weights(dims, parts))
    got = pu.gpu_act(net, cfg, inp)
    np.testing.assert_allclose(got["h_out"], inp["h_in"], atol=1e-6)
    net.close()
    # exact ties: lowest index wins; an unavailable leader is skipped
    parts = dict(zero)
    parts["b2"] = np.array([0.1, 0.9, 0.3, 0.9, -1.0, 0.9, 0, 0, 0])
    net, w = make_net(cfg, weights=wl.pack_weights(dims, parts))
    inp["epsilon"] = 0.0
    got = pu.gpu_act(net, cfg, inp)
    np.testing.assert_array_equal(got["action"], oracle_act(cfg, w, inp)["action"])
    none = dict(inp); none["avail"] = np.zeros_like(inp["avail"])
    for eps in (0.0, 1.0):
        none["epsilon"] = eps
        assert (pu.gpu_act(net, cfg, none)["action"] == 0).all()      # nothing available -> action 0
    net.close()


def test_act_step_episode_loop_feeds_hidden_state_back():
    cfg = wl.config(0)
    N, D, A, H = wl.dims(cfg)
    net, w = make_net(cfg)
    E, T = 5, cfg["T"]
    u = wl.make_unroll_inputs(cfg, B=E)
    h_gpu = np.zeros((E, N, H), np.float32)
    h_ref = np.zeros((E, N, H))
    for t in range(T + 1):
        inp = dict(obs=u["obs"][:, t], avail=u["avail"][:, t], reset=np.full(E, t == 0, np.uint8),
                   step_t=np.full(E, t, np.int32), epsilon=0.3, seed=99)
        ref = oracle_act(cfg, w, dict(inp, h_in=h_ref))
        got = pu.gpu_act(net, cfg, dict(inp, h_in=h_gpu))
        pu.compare_act(cfg, inp, got, ref, 1e-4)
        h_gpu, h_ref = got["h_out"], ref["h_out"]
    net.close()


def test_act_step_is_deterministic_and_isolated():
    cfg = wl.config(1)
    net, _ = make_net(cfg)
    inp = wl.make_act_inputs(cfg, E=64)
    a = pu.gpu_act(net, cfg, inp)
    b = pu.gpu_act(net, cfg, inp)
    for k in ("q", "h_out", "action"):
        np.testing.assert_array_equal(a[k], b[k])
    mod = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in inp.items()}
    mod["obs"][5] += 1.0
    mod["h_in"][5] *= -1.0
    c = pu.gpu_act(net, cfg, mod)
    others = np.arange(64) != 5
    for k in ("q", "h_out", "action"):
        np.testing.assert_array_equal(c[k][others], a[k][others])
    assert (c["q"][5] != a["q"][5]).any()
    # a sub-batch of the first environments gives the same rows
    sub = {k: (v[:17] if isinstance(v, np.ndarray) else v) for k, v in inp.items()}
    d = pu.gpu_act(net, cfg, sub)
    np.testing.assert_array_equal(d["action"], a["action"][:17])
    np.testing.assert_allclose(d["q"], a["q"][:17], atol=1e-6)
    net.close()


# ------------------------------------------------------------------ unroll + TD
@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
@pytest.mark.parametrize("ci", [0, 1, 2, 3])
def test_unroll_td_full_config(ci, path):
    cfg = wl.config(ci)
    tol = pu.TOL[cfg["dtype"]]
    online, w_on = make_net(cfg, 0)
    target, w_tg = make_net(cfg, 1)
    online.set_kernels(path)
    u = wl.make_unroll_inputs(cfg)
    got = pu.gpu_unroll(online, target, cfg, u)
    ref = oracle_unroll(cfg, w_on, w_tg, u)
    worst = pu.compare_unroll(got, ref, tol)
    pad = u["filled"] == 0
    for k in ("q_taken", "next_max", "td_target"):
        assert (got[k][pad] == 0.0).all()                 # padded transitions are exactly zero
    got1 = pu.gpu_unroll(online, None, cfg, u, want_q_all=False)     # target == online, no q_all
    ref1 = oracle_unroll(cfg, w_on, None, u)
    worst1 = pu.compare_unroll(got1, ref1, tol)
    print(f"cfg{ci}: two nets maxerr={worst:.3e}, one net maxerr={worst1:.3e}")
    online.close(); target.close()


_CFG4_ORACLE = {}


def cfg4_oracle_unroll():
    """The oracle's unroll of the whole scale-up batch (all 2,048 rows, both networks, every Q value), computed
    once per session: a few seconds on the host's cores."""
    if not _CFG4_ORACLE:
        cfg = wl.config(4)
        w_on = pu.oracle_weights(cfg, wl.make_weights(cfg, 0))
        w_tg = pu.oracle_weights(cfg, wl.make_weights(cfg, 1))
        u = wl.make_unroll_inputs(cfg)
        _CFG4_ORACLE.update(u=u, ref=oracle_unroll(cfg, w_on, w_tg, u))
    return _CFG4_ORACLE["u"], _CFG4_ORACLE["ref"]


@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
def test_unroll_td_full_config_4_every_row(path):
    """The scale-up workload at full size, in the launch configuration the benchmark times: every output of every
    (episode, agent) row against the oracle."""
    cfg = wl.config(4)
    tol = pu.TOL[cfg["dtype"]]
    online, w_on = make_net(cfg, 0)
    target, w_tg = make_net(cfg, 1)
    online.set_kernels(path)
    u, ref = cfg4_oracle_unroll()
    got = pu.gpu_unroll(online, target, cfg, u)
    worst = pu.compare_unroll(got, ref, tol)
    print(f"cfg4: all {cfg['B'] * cfg['N']} rows, maxerr={worst:.3e}")
    pad = u["filled"] == 0
    for k in ("q_taken", "next_max", "td_target"):
        assert (got[k][pad] == 0.0).all()
    g = np.float32(u["gamma"])
    keep = (1.0 - u["terminated"].astype(np.float32))[..., None]
    expect = (u["reward"][..., None] + g * keep * got["next_max"]) * u["filled"][..., None]
    np.testing.assert_allclose(got["td_target"], expect, atol=1e-5)
    taken = np.take_along_axis(got["q_all"][:, :-1], u["actions"][..., None].astype(np.int64), -1)[..., 0]
    np.testing.assert_array_equal(got["q_taken"], taken * u["filled"][..., None])
    online.close(); target.close()


@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
@pytest.mark.parametrize("ci,B,T", [(0, 1, 1), (0, 3, 7), (1, 5, 9), (2, 7, 3), (3, 33, 5), (4, 2, 6)])
def test_unroll_td_ragged_sizes(ci, B, T, path):
    cfg = wl.config(ci)
    online, w_on = make_net(cfg, 0)
    target, w_tg = make_net(cfg, 1)
    online.set_kernels(path)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    got = pu.gpu_unroll(online, target, cfg, u)
    ref = oracle_unroll(cfg, w_on, w_tg, u)
    pu.compare_unroll(got, ref, pu.TOL[cfg["dtype"]])
    online.close(); target.close()


def test_unroll_td_special_cases():
    cfg = wl.config(0)
    online, w_on = make_net(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=6, T=11)
    u0 = dict(u, gamma=0.0)
    got = pu.gpu_unroll(online, None, cfg, u0)
    expect = np.broadcast_to((u["reward"] * u["filled"])[..., None], got["td_target"].shape)
    np.testing.assert_array_equal(got["td_target"], expect)              # gamma = 0: y = r
    u1 = dict(u, terminated=np.ones_like(u["terminated"]))
    got = pu.gpu_unroll(online, None, cfg, u1)
    np.testing.assert_array_equal(got["td_target"], expect)              # terminated: y = r
    u2 = dict(u, avail=np.zeros_like(u["avail"]))
    got = pu.gpu_unroll(online, None, cfg, u2)
    assert (got["next_max"] == 0.0).all()                                 # nothing available: bootstrap 0
    online.close()


def test_unroll_matches_iterated_act_step_on_gpu():
    cfg = wl.config(1)
    N, D, A, H = wl.dims(cfg)
    net, _ = make_net(cfg)
    B, T = 6, 20
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    got = pu.gpu_unroll(net, None, cfg, u)
    h = np.zeros((B, N, H), np.float32)
    for t in range(T + 1):
        inp = dict(obs=u["obs"][:, t], avail=u["avail"][:, t], h_in=h, reset=np.full(B, t == 0, np.uint8),
                   step_t=np.full(B, t, np.int32), epsilon=0.0, seed=1)
        a = pu.gpu_act(net, cfg, inp)
        np.testing.assert_allclose(a["q"], got["q_all"][:, t], atol=2e-5)
        h = a["h_out"]
    net.close()


# ------------------------------------------------------------------ boundary behaviour on the device
def test_empty_batches_and_argument_errors():
    cfg = wl.config(0)
    N, D, A, H = wl.dims(cfg)
    net, _ = make_net(cfg)
    other, _ = make_net(wl.config(1))
    lib = binding.load()
    import ctypes
    hp = ctypes.c_void_p(net.handle)
    assert lib.marl_act_step(hp, 0, None, None, None, None, None, 0.1, 0, None, None, None, None) == 0
    assert lib.marl_unroll_td(hp, hp, 0, 5, None, None, None, None, None, None, 0.9, None, None, None, None, None) == 0
    assert lib.marl_act_step(hp, -1, None, None, None, None, None, 0.1, 0, None, None, None, None) == -2
    assert lib.marl_act_step(hp, 4, None, None, None, None, None, 0.1, 0, None, None, None, None) == -1
    assert lib.marl_act_step(hp, 4, None, None, None, None, None, 1.5, 0, None, None, None, None) == -5
    assert lib.marl_act_step(hp, 4, None, None, None, None, None, float("nan"), 0, None, None, None, None) == -5
    assert lib.marl_unroll_td(hp, hp, 2, 0, None, None, None, None, None, None, 0.9, None, None, None, None, None) == -2
    assert lib.marl_unroll_td(hp, hp, 2, 3, None, None, None, None, None, None, -0.1, None, None, None, None, None) == -5
    assert lib.marl_unroll_td(hp, ctypes.c_void_p(other.handle), 2, 3, None, None, None, None, None, None, 0.9,
                              None, None, None, None, None) == -4
    d = binding.Desc()
    assert lib.marl_qnet_get_desc(hp, ctypes.byref(d)) == 0 and (d.n_agents, d.obs_dim, d.n_actions, d.hidden) == (N, D, A, H)
    with pytest.raises(ValueError):
        net.act_step(torch.zeros(2, N, D), torch.zeros(2, N, A, dtype=torch.uint8), torch.zeros(2, N, H), None,
                     torch.zeros(2, dtype=torch.int32), 0.0, 0, torch.zeros(2, N, H), torch.zeros(2, N, dtype=torch.int32))
    net.close(); other.close()


# ------------------------------------------------------------------ kernel families
@pytest.mark.parametrize("D,dtype,fused", [(320, "bf16", True), (352, "bf16", False), (160, "fp32", True), (176, "fp32", False)])
def test_kernel_family_follows_the_network_shape(D, dtype, fused):
    """Networks at and just past the fused kernels' limits: the library picks the family that
    fits, both stay inside the tolerance, and forcing the fused family on a misfit is refused."""
    base = wl.config(4 if dtype == "bf16" else 2)
    cfg = dict(base, D=D, dtype=dtype, E=6, B=3, T=7)
    net, w = make_net(cfg)
    target, w_tg = make_net(cfg, 1)
    want = binding.KERNELS_FUSED16 if fused else binding.KERNELS_TILE32
    assert net.kernels_in_use(binding.ENTRY_ACT_STEP) == want
    assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == want
    if not fused:
        with pytest.raises(binding.MarlError) as err:
            net.set_kernels(binding.KERNELS_FUSED16)
        assert err.value.status == -2                     # MARL_ERR_BAD_DIM
    with pytest.raises(binding.MarlError):
        net.set_kernels(7)
    inp = wl.make_act_inputs(cfg)
    pu.compare_act(cfg, inp, pu.gpu_act(net, cfg, inp), oracle_act(cfg, w, inp), pu.TOL[dtype])
    u = wl.make_unroll_inputs(cfg)
    pu.compare_unroll(pu.gpu_unroll(net, target, cfg, u), oracle_unroll(cfg, w, w_tg, u), pu.TOL[dtype])
    net.set_kernels(binding.KERNELS_TILE32)
    assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == binding.KERNELS_TILE32
    pu.compare_unroll(pu.gpu_unroll(net, target, cfg, u), oracle_unroll(cfg, w, w_tg, u), pu.TOL[dtype])
    net.close(); target.close()


# ------------------------------------------------------------------ weight refresh
@pytest.mark.parametrize("ci", [1, 4])
def test_set_weights_is_ordered_on_the_stream(ci):
    """New parameters published in place: calls enqueued before the refresh see the old network,
    calls after it the new one, with no synchronisation in between; a second refresh right after
    the first does not disturb it."""
    cfg = dict(wl.config(ci), E=64, B=4, T=9)
    w0, w1, w2 = (wl.make_weights(cfg, s) for s in (0, 1, 2))
    net = binding.QNet(wl.dims(cfg), w0, cfg["dtype"])
    inp = wl.make_act_inputs(cfg)
    u = wl.make_unroll_inputs(cfg)
    tol = pu.TOL[cfg["dtype"]]
    N, D, A, H = wl.dims(cfg)
    d = pu.to_dev(inp, ["obs", "avail", "h_in", "reset", "step_t"])
    outs = []
    for w in (None, w1, w2):
        if w is not None:
            net.set_weights(w)
        h_out = torch.empty(cfg["E"], N, H, device="cuda")
        act = torch.empty(cfg["E"], N, dtype=torch.int32, device="cuda")
        q = torch.empty(cfg["E"], N, A, device="cuda")
        net.act_step(d["obs"], d["avail"], d["h_in"], d["reset"], d["step_t"], inp["epsilon"], inp["seed"], h_out, act, q)
        outs.append((h_out, act, q))
    torch.cuda.synchronize()
    for (h_out, act, q), w in zip(outs, (w0, w1, w2)):
        ref = oracle_act(cfg, pu.oracle_weights(cfg, w), inp)
        got = {"h_out": h_out.cpu().numpy(), "action": act.cpu().numpy(), "q": q.cpu().numpy()}
        pu.compare_act(cfg, inp, got, ref, tol)
    ref = oracle_unroll(cfg, pu.oracle_weights(cfg, w2), None, u)
    pu.compare_unroll(pu.gpu_unroll(net, None, cfg, u), ref, tol)
    with pytest.raises(binding.MarlError):
        net.set_weights(w0[:-1])
    net.close()


# ------------------------------------------------------------------ shapes at the edges of the supported range
ODD_SHAPES = [
    # N, D, A, H, dtype
    (1, 1, 1, 64, "fp32"),          # one agent, one observation value, one action
    (2, 7, 3, 64, "fp32"),          # fewer than four actions (byte-wise availability path)
    (3, 31, 4, 64, "bf16"),
    (5, 32, 17, 64, "fp32"),        # exactly one full k-step; two action blocks, ragged
    (7, 33, 33, 128, "bf16"),       # one value past a k-step; three action blocks
    (64, 64, 64, 128, "bf16"),      # the maxima of N and A
    (4, 97, 48, 64, "bf16"),
    (6, 160, 16, 64, "fp32"),       # the largest obs_dim the fused fp32 kernels take
    (9, 320, 40, 128, "bf16"),      # the largest obs_dim the fused bf16 kernels take
]


@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
@pytest.mark.parametrize("shape", ODD_SHAPES, ids=lambda s: "N%d_D%d_A%d_H%d_%s" % s)
def test_odd_shapes(shape, path):
    N, D, A, H, dtype = shape
    cfg = dict(wl.config(0), N=N, D=D, A=A, H=H, dtype=dtype, E=11, B=5, T=6)
    tol = pu.TOL[dtype]
    if path == binding.KERNELS_FUSED16 and A < 4:
        # the fused decision step reads availability four bytes at a time: the fused family as a
        # whole is refused, and left to itself the library mixes the two
        net, w = make_net(cfg)
        with pytest.raises(binding.MarlError) as err:
            net.set_kernels(binding.KERNELS_FUSED16)
        assert err.value.status == -2                     # MARL_ERR_BAD_DIM
        assert net.kernels_in_use(binding.ENTRY_ACT_STEP) == binding.KERNELS_TILE32
        assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == binding.KERNELS_FUSED16
    else:
        net, w = make_net(cfg, kernels=path)
    target, w_tg = make_net(cfg, 1)
    for eps in (0.0, 1.0):
        inp = wl.make_act_inputs(cfg, stream=3)
        inp["epsilon"] = eps
        got = pu.gpu_act(net, cfg, inp)
        pu.compare_act(cfg, inp, got, oracle_act(cfg, w, inp), tol)
        assert np.take_along_axis(inp["avail"], got["action"][..., None].astype(np.int64), -1).all()
    u = wl.make_unroll_inputs(cfg)
    pu.compare_unroll(pu.gpu_unroll(net, target, cfg, u), oracle_unroll(cfg, w, w_tg, u), tol)
    net.close(); target.close()


@pytest.mark.parametrize("H,dtype", [(64, "fp32"), (64, "bf16"), (128, "bf16")])
@pytest.mark.parametrize("D", [1, 7, 8, 9, 39, 63, 65, 96, 127, 129, 161, 193, 225, 257, 289, 313])
def test_unroll_observation_widths(D, H, dtype):
    """The fused unroll reads the last eight observations of a row from the row's end and runs a number of k-steps that may be
    rounded up: widths around eight, around whole k-steps and in every such number; 19 rows, T odd and even."""
    if dtype == "fp32" and D > 160:
        pytest.skip("wider than the fused kernels take in two planes")
    cfg = dict(wl.config(0), N=19, D=D, A=5, H=H, dtype=dtype, B=1, T=4 + D % 2)
    net, w = make_net(cfg)
    target, w_tg = make_net(cfg, 1)
    assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == binding.KERNELS_FUSED16
    u = wl.make_unroll_inputs(cfg)
    pu.compare_unroll(pu.gpu_unroll(net, target, cfg, u), oracle_unroll(cfg, w, w_tg, u), pu.TOL[dtype])
    net.close(); target.close()


# Shapes the descriptor admits that only the tiled kernels take: fp32 weights with 128 hidden units, and
# observations up to the widest the library accepts.
TILED_ONLY_SHAPES = [
    # N, D, A, H, dtype
    (4, 40, 12, 128, "fp32"),
    (32, 300, 40, 128, "fp32"),     # the scale-up network with fp32 weights
    (3, 1024, 40, 128, "bf16"),     # the widest observation
    (2, 1024, 9, 64, "fp32"),
    (2, 1024, 64, 128, "fp32"),     # every maximum at once but the agent count
    (64, 1000, 5, 64, "bf16"),      # a one-hot identity that straddles a 32-wide k-step at the end of a wide row
]


@pytest.mark.parametrize("shape", TILED_ONLY_SHAPES, ids=lambda s: "N%d_D%d_A%d_H%d_%s" % s)
def test_shapes_only_the_tiled_kernels_take(shape):
    N, D, A, H, dtype = shape
    cfg = dict(wl.config(0), N=N, D=D, A=A, H=H, dtype=dtype, E=37, B=5, T=6)
    tol = pu.TOL[dtype]
    net, w = make_net(cfg)
    target, w_tg = make_net(cfg, 1)
    assert net.kernels_in_use(binding.ENTRY_ACT_STEP) == binding.KERNELS_TILE32
    assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == binding.KERNELS_TILE32
    for other in (binding.KERNELS_FUSED16, binding.KERNELS_STREAM16):
        with pytest.raises(binding.MarlError) as err:
            net.set_kernels(other)
        assert err.value.status == -2                     # MARL_ERR_BAD_DIM
    for eps in (0.0, 0.3):
        inp = wl.make_act_inputs(cfg, stream=5)
        inp["epsilon"] = eps
        got = pu.gpu_act(net, cfg, inp)
        pu.compare_act(cfg, inp, got, oracle_act(cfg, w, inp), tol)
        assert np.take_along_axis(inp["avail"], got["action"][..., None].astype(np.int64), -1).all()
    u = wl.make_unroll_inputs(cfg)
    worst = pu.compare_unroll(pu.gpu_unroll(net, target, cfg, u), oracle_unroll(cfg, w, w_tg, u), tol)
    print(shape, f"unroll maxerr={worst:.3e}")
    net.close(); target.close()


# ------------------------------------------------------------------ HIP graph capture
@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
def test_calls_replay_from_a_hip_graph(path):
    """One decision step and one unroll captured into a HIP graph (after one eager call, which
    sizes whatever the handle caches) and replayed three times on fresh input values, with eager
    work and synchronisation between the replays: every replay matches the eager call on the same
    values bit for bit, and the first also matches the oracle."""
    cfg = dict(wl.config(1), E=96, B=6, T=11)
    N, D, A, H = wl.dims(cfg)
    tol = pu.TOL[cfg["dtype"]]
    net, w = make_net(cfg, kernels=path)
    target, w_tg = make_net(cfg, 1, kernels=path)
    inputs = [(wl.make_act_inputs(cfg, stream=s), wl.make_unroll_inputs(cfg, stream=s)) for s in range(3)]
    a_keys, u_keys = ["obs", "avail", "h_in", "reset", "step_t"], ["obs", "avail", "actions", "reward", "terminated", "filled"]
    a = pu.to_dev(inputs[0][0], a_keys)
    u = pu.to_dev(inputs[0][1], u_keys)
    E, B, T = cfg["E"], cfg["B"], cfg["T"]
    out = dict(h=torch.empty(E, N, H, device="cuda"), act=torch.empty(E, N, dtype=torch.int32, device="cuda"),
               q=torch.empty(E, N, A, device="cuda"), u=[torch.empty(B, T, N, device="cuda") for _ in range(3)])

    def calls():
        net.act_step(a["obs"], a["avail"], a["h_in"], a["reset"], a["step_t"], inputs[0][0]["epsilon"],
                     inputs[0][0]["seed"], out["h"], out["act"], out["q"])
        net.unroll_td(target, u["obs"], u["avail"], u["actions"], u["reward"], u["terminated"], u["filled"],
                      inputs[0][1]["gamma"], *out["u"])

    def snapshot():
        torch.cuda.synchronize()
        return [out["h"].clone(), out["act"].clone(), out["q"].clone()] + [t.clone() for t in out["u"]]

    calls()                                   # eager: caches are sized, launch attributes set
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            calls()
    torch.cuda.synchronize()
    for r, (ai, ui) in enumerate(inputs):
        for k in a_keys:
            a[k].copy_(torch.from_numpy(np.ascontiguousarray(ai[k])))
        for k in u_keys:
            u[k].copy_(torch.from_numpy(np.ascontiguousarray(ui[k])))
        calls()
        eager = snapshot()
        for t in [out["h"], out["q"]] + out["u"]:
            t.fill_(float("nan"))
        out["act"].fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        replayed = snapshot()
        for e, g in zip(eager, replayed):
            assert torch.equal(e, g), f"replay {r} differs from the eager call"
        if r == 0:
            got = {"h_out": replayed[0].cpu().numpy(), "action": replayed[1].cpu().numpy(), "q": replayed[2].cpu().numpy()}
            pu.compare_act(cfg, ai, got, oracle_act(cfg, w, ai), tol)
    net.close(); target.close()


# ------------------------------------------------------------------ asynchronous sub-batch
@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
@pytest.mark.parametrize("ci,n_listed", [(0, 3), (1, 100), (3, 1), (3, 777), (4, 50), (4, 1024), (2, 512)])
def test_indexed_decision_step_serves_only_the_listed_environments(ci, n_listed, path):
    """A random subset of the environments, in random order: their rows get exactly what the oracle
    gives them in a step over all environments (same random-number key, which uses the environment's
    own index), every other row of every output keeps its previous contents, and the hidden-state
    table may be updated in place."""
    cfg = dict(wl.config(ci))
    cfg["E"] = min(cfg["E"], 1024)
    tol = pu.TOL[cfg["dtype"]]
    N, D, A, H = wl.dims(cfg)
    net, w = make_net(cfg, kernels=path)
    inp = wl.make_act_inputs(cfg)
    E = cfg["E"]
    listed = np.random.default_rng(ci).permutation(E)[:n_listed].astype(np.int32)
    ref = oracle_act(cfg, w, inp)
    d = pu.to_dev(inp, ["obs", "avail", "h_in", "reset", "step_t"])
    idx = torch.from_numpy(listed).cuda()
    h_table = d["h_in"].clone()                       # updated in place
    action = torch.full((E, N), -7, dtype=torch.int32, device="cuda")
    q = torch.full((E, N, A), -123.0, device="cuda")
    net.act_step_indexed(idx, d["obs"], d["avail"], h_table, d["reset"], d["step_t"], inp["epsilon"], inp["seed"],
                         h_table, action, q)
    torch.cuda.synchronize()
    served = np.zeros(E, bool); served[listed] = True
    got = {"h_out": h_table.cpu().numpy(), "action": action.cpu().numpy(), "q": q.cpu().numpy()}
    sub = lambda x: {k: v[served] for k, v in x.items()}
    pu.compare_act(cfg, {k: (inp[k][served] if isinstance(inp[k], np.ndarray) else inp[k]) for k in inp}, sub(got),
                   {k: v[served] for k, v in ref.items()}, tol)
    np.testing.assert_array_equal(got["h_out"][~served], inp["h_in"][~served])
    assert (got["action"][~served] == -7).all() and (got["q"][~served] == -123.0).all()
    with pytest.raises(binding.MarlError) as err:
        binding.check(binding.load().marl_act_step_indexed(net.handle, E, None, E + 1, *([None] * 5), 0.0, 0, None, None, None, None))
    assert err.value.status == -2
    net.close()


# ------------------------------------------------------------------ replay pool read in place
@pytest.mark.parametrize("ci,pool,B", [(0, 9, 4), (1, 40, 24), (3, 50, 70), (4, 12, 7)])
def test_indexed_unroll_reads_the_batch_from_a_pool(ci, pool, B):
    """B episodes drawn with replacement from a pool of episodes: the call that reads the pool in place
    gives, per batch position, exactly what the oracle gives on the gathered batch (and bit for bit
    what the library's own packed-batch call gives)."""
    cfg = dict(wl.config(ci), T=min(wl.config(ci)["T"], 25))
    tol = pu.TOL[cfg["dtype"]]
    N, D, A, H = wl.dims(cfg)
    T = cfg["T"]
    net, w = make_net(cfg)
    target, w_tg = make_net(cfg, 1)
    assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == binding.KERNELS_FUSED16
    u = wl.make_unroll_inputs(cfg, B=pool)
    pick = np.random.default_rng(ci + 10).integers(0, pool, B).astype(np.int32)
    keys = ["obs", "avail", "actions", "reward", "terminated", "filled"]
    packed = dict(u, **{k: np.ascontiguousarray(u[k][pick]) for k in keys})
    d = pu.to_dev(u, keys)
    outs = {k: torch.full((B, T, N), float("nan"), device="cuda") for k in ("q_taken", "next_max", "td_target")}
    q_all = torch.full((B, T + 1, N, A), float("nan"), device="cuda")
    net.unroll_td_indexed(target, torch.from_numpy(pick).cuda(), d["obs"], d["avail"], d["actions"], d["reward"],
                          d["terminated"], d["filled"], u["gamma"], outs["q_taken"], outs["next_max"], outs["td_target"], q_all)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in outs.items()}
    got["q_all"] = q_all.cpu().numpy()
    pu.compare_unroll(got, oracle_unroll(cfg, w, w_tg, packed), tol)
    same = pu.gpu_unroll(net, target, cfg, packed)
    for k in got:
        np.testing.assert_array_equal(got[k], same[k])
    lib, vp = binding.load(), ctypes.c_void_p
    args = lambda pool_n, index, b: (vp(net.handle), vp(target.handle), pool_n, index, b, T, vp(d["obs"].data_ptr()),
                                     vp(d["avail"].data_ptr()), vp(d["actions"].data_ptr()), vp(d["reward"].data_ptr()),
                                     vp(d["terminated"].data_ptr()), vp(d["filled"].data_ptr()), 0.9, vp(outs["q_taken"].data_ptr()),
                                     vp(outs["next_max"].data_ptr()), vp(outs["td_target"].data_ptr()), None, None)
    index_ptr = vp(torch.from_numpy(pick).cuda().data_ptr())
    assert lib.marl_unroll_td_indexed(*args(pool, index_ptr, 0)) == 0         # empty batch: nothing to do
    assert lib.marl_unroll_td_indexed(*args(0, index_ptr, B)) == -2           # empty pool
    assert lib.marl_unroll_td_indexed(*args(pool, None, B)) == -1             # no index
    torch.cuda.synchronize()
    # the two-kernel family reads the pool in place as well
    net.set_kernels(binding.KERNELS_TILE32)
    for t in list(outs.values()) + [q_all]:
        t.fill_(float("nan"))
    net.unroll_td_indexed(target, torch.from_numpy(pick).cuda(), d["obs"], d["avail"], d["actions"], d["reward"],
                          d["terminated"], d["filled"], u["gamma"], outs["q_taken"], outs["next_max"], outs["td_target"], q_all)
    torch.cuda.synchronize()
    got32 = {k: v.cpu().numpy() for k, v in outs.items()}
    got32["q_all"] = q_all.cpu().numpy()
    pu.compare_unroll(got32, oracle_unroll(cfg, w, w_tg, packed), tol)
    net.close(); target.close()


# ------------------------------------------------------------------ double-estimator target
def run_double(net, target, cfg, u, d, index=None, want_q_all=True):
    N, D, A, H = wl.dims(cfg)
    T = u["actions"].shape[1]
    B = u["actions"].shape[0] if index is None else index.shape[0]
    outs = {k: torch.full((B, T, N), float("nan"), device="cuda") for k in ("q_taken", "next_max", "td_target")}
    nxt = torch.full((B, T, N), -9, dtype=torch.int32, device="cuda")
    q_all = torch.full((B, T + 1, N, A), float("nan"), device="cuda") if want_q_all else None
    net.unroll_td_double(target, d["obs"], d["avail"], d["actions"], d["reward"], d["terminated"], d["filled"],
                         u["gamma"], outs["q_taken"], outs["next_max"], outs["td_target"], nxt, q_all,
                         None if index is None else torch.from_numpy(index).cuda())
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in outs.items()}
    got["next_action"] = nxt.cpu().numpy()
    got["q_all"] = None if q_all is None else q_all.cpu().numpy()
    return got


def compare_double(cfg, u, got, w_on, w_tg, tol):
    """u: the batch as the oracle sees it.  The index is exact wherever the online network's best
    available value at t+1 leads by more than tol; inside a near-tie any available action within
    tol of the best passes.  The values are those of the target network at the index returned."""
    dims = wl.dims(cfg)
    ref = orc.unroll_td_double(dims, w_on, w_tg, u["obs"], u["avail"], u["actions"], u["reward"], u["terminated"],
                               u["filled"], u["gamma"])
    q_tg = orc.unroll_td(dims, w_tg, None, u["obs"], u["avail"], u["actions"], u["reward"], u["terminated"],
                         u["filled"], u["gamma"])["q_all"]
    assert np.abs(got["q_taken"] - ref["q_taken"]).max() <= tol
    if got["q_all"] is not None:
        assert np.abs(got["q_all"] - ref["q_all"]).max() <= tol
    avail = u["avail"][:, 1:] != 0
    masked = np.where(avail, ref["q_all"][:, 1:], -np.inf)
    top = np.sort(masked, -1)
    best = top[..., -1]
    second = top[..., -2] if masked.shape[-1] > 1 else np.full(best.shape, -np.inf)
    none = ~avail.any(-1)
    with np.errstate(invalid="ignore"):
        clear = ((best - second) > tol) | none
    a = got["next_action"]
    assert (a[clear] == ref["next_action"][clear]).all(), "index mismatch outside near-ties"
    assert (a[none] == -1).all()
    tie = ~clear
    if tie.any():
        chosen = np.take_along_axis(masked[tie], a[tie].astype(np.int64)[:, None], -1)[:, 0]
        assert (chosen >= best[tie] - tol).all(), "near-tie index is not one of the leaders"
    value = np.take_along_axis(q_tg[:, 1:], np.maximum(a, 0).astype(np.int64)[..., None], -1)[..., 0]
    value = np.where(none, 0.0, value)
    f = (u["filled"] != 0).astype(np.float64)[..., None]
    keep = 1.0 - (u["terminated"] != 0).astype(np.float64)[..., None]
    y = u["reward"].astype(np.float64)[..., None] + float(np.float32(u["gamma"])) * keep * value
    assert np.abs(got["next_max"] - f * value).max() <= tol
    assert np.abs(got["td_target"] - f * y).max() <= tol
    assert (a[clear] == ref["next_action"][clear]).mean() == 1.0
    return int(tie.sum())


@pytest.mark.parametrize("path", PATHS, ids=PATH_IDS)
@pytest.mark.parametrize("ci,B,T", [(0, 32, 25), (1, 13, 9), (2, 7, 12), (3, 33, 5), (4, 5, 11)])
def test_double_estimator_target(ci, B, T, path):
    cfg = dict(wl.config(ci), B=B, T=T)
    tol = pu.TOL[cfg["dtype"]]
    net, w = make_net(cfg, kernels=path)
    target, w_tg = make_net(cfg, 1, kernels=path)
    assert net.kernels_in_use(binding.ENTRY_UNROLL_TD) == path
    keys = ["obs", "avail", "actions", "reward", "terminated", "filled"]
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    u["avail"][0, 2, 0, :] = 0                                 # a row with nothing available: index -1, value 0
    d = pu.to_dev(u, keys)
    got = run_double(net, target, cfg, u, d)
    ties = compare_double(cfg, u, got, w, w_tg, tol)
    assert ties < (0.05 if cfg["dtype"] == "fp32" else 0.25) * got["next_action"].size     # the exact check covers the rest
    # it is not the plain target: somewhere the target network prefers another action
    plain = pu.gpu_unroll(net, target, cfg, u)
    assert (got["next_max"] <= plain["next_max"] + 2 * tol).all() and (got["next_max"] < plain["next_max"]).any()
    np.testing.assert_array_equal(got["q_taken"], plain["q_taken"])
    np.testing.assert_array_equal(got["q_all"], plain["q_all"])
    # one handle on both sides: the plain target's numbers, bit for bit
    one = run_double(net, None, cfg, u, d, want_q_all=False)
    plain_one = pu.gpu_unroll(net, None, cfg, u, want_q_all=False)
    for k in ("q_taken", "next_max", "td_target"):
        np.testing.assert_array_equal(one[k], plain_one[k])
    # the batch read in place from a pool
    pick = np.random.default_rng(ci + 20).integers(0, B, 6).astype(np.int32)
    packed = dict(u, **{k: np.ascontiguousarray(u[k][pick]) for k in keys})
    pooled = run_double(net, target, cfg, u, d, index=pick)
    compare_double(cfg, packed, pooled, w, w_tg, tol)
    for k in ("q_taken", "next_max", "td_target", "next_action", "q_all"):
        np.testing.assert_array_equal(pooled[k], got[k][pick])
    # a missing index array is refused before anything is launched
    lib, vp = binding.load(), ctypes.c_void_p
    rc = lib.marl_unroll_td_double(vp(net.handle), vp(target.handle), B, None, B, T, vp(d["obs"].data_ptr()),
                                   vp(d["avail"].data_ptr()), vp(d["actions"].data_ptr()), vp(d["reward"].data_ptr()),
                                   vp(d["terminated"].data_ptr()), vp(d["filled"].data_ptr()), 0.9,
                                   vp(d["obs"].data_ptr()), vp(d["obs"].data_ptr()), vp(d["obs"].data_ptr()), None, None, None)
    assert rc == -1
    net.close(); target.close()


# ------------------------------------------------------------------ measurement aids
def test_probes_copy_what_they_read_and_check_their_arguments():
    lib, vp = binding.load(), ctypes.c_void_p
    src = torch.arange(4 * 100003, dtype=torch.float32, device="cuda")      # a vector count no grid stride divides
    dst = torch.zeros_like(src)
    sink = torch.zeros(1, device="cuda")
    assert binding.marl_probe_stream(src, dst, sink) == 2 * src.numel() * 4
    assert binding.marl_probe_stream(src, None, sink) == src.numel() * 4
    torch.cuda.synchronize()
    assert torch.equal(dst, src) and float(sink) == 0.0
    flops = binding.marl_probe_mfma(10, sink)
    torch.cuda.synchronize()
    assert flops == torch.cuda.get_device_properties(0).multi_processor_count * 2 * 4 * 10 * 8 * 2 * 16 * 16 * 32
    assert float(sink) == 0.0
    p = vp(src.data_ptr())
    assert lib.marl_probe_stream(p, None, 24, vp(sink.data_ptr()), None) == -2          # not a multiple of 16
    assert lib.marl_probe_stream(vp(src.data_ptr() + 4), None, 32, vp(sink.data_ptr()), None) == -5
    assert lib.marl_probe_stream(None, None, 32, vp(sink.data_ptr()), None) == -1
    assert lib.marl_probe_mfma(0, vp(sink.data_ptr()), ctypes.byref(ctypes.c_double()), None) == -2
