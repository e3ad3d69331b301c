"""An infinite observation in a bf16 network's unroll reaches the first layer once, with its own weight: the oracle's Q values,
and those of the fused decision step, slot by slot.

The weights keep an infinity meaningful: W1 positive, so that every x of the row is +inf; each row of W_ih of one sign, so that
the gates saturate and the state stays finite.  Where the row's length is not a whole number of k-steps of 32, the decision step's
loader has the row's last value also in the places past the end, at zero weights, and so has the unroll's for rows of less than
eight: an infinity there makes NaN of the sums and 0 of x.  Such a row is compared between those two only, or with the oracle only."""
import numpy as np
import pytest
import torch

from paper_2205_05248_amd import binding, workloads as wl
import parity_util as pu
import test_gpu_bptt as bptt
from test_gpu_parity import oracle_unroll

pytestmark = pytest.mark.gpu
TOL = pu.TOL["bf16"]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


def saturating_weights(cfg):
    w = wl.make_weights(cfg, 0).copy()
    at = {k: w[a:b].reshape(shp) for k, (a, b, shp) in wl.weight_slices(*wl.dims(cfg)).items()}
    at["W1"][:] = 0.2 * np.abs(at["W1"]) + 1e-3
    at["W_ih"][:] = (np.abs(at["W_ih"]) + 1e-3) * np.where(np.arange(len(at["W_ih"])) % 3 == 1, -1, 1)[:, None]
    return w


# ends of rows inside, at and past a group of eight and a k-step; numbers of k-steps as they are (1 to 4) and rounded up (5, 7, 9)
@pytest.mark.parametrize("H", [64, 128])
@pytest.mark.parametrize("D", [5, 8, 13, 32, 33, 40, 63, 96, 100, 128, 129, 160, 161, 192, 223, 225, 256, 257, 288, 300, 320])
def test_an_infinite_observation_counts_once(D, H):
    at = sorted({p for p in (0, D // 2, D - 9, D - 8, D - 7, D - 3, D - 2, D - 1) if 0 <= p < D})
    cfg = dict(wl.config(0), N=len(at) + 1, D=D, A=6, H=H, dtype="bf16", B=2, T=4)
    N, slot, T = cfg["N"], 2, cfg["T"]
    w = saturating_weights(cfg)
    u = wl.make_unroll_inputs(cfg)
    for n, p in enumerate(at):                       # (the last agent's rows stay finite)
        u["obs"][0, slot, n, p] = np.inf
    u["obs"][1, 1, 0, at[len(at) // 2]] = -np.inf
    net = binding.QNet(wl.dims(cfg), w, "bf16")
    net.set_kernels(binding.KERNELS_FUSED16)
    got = pu.gpu_unroll(net, None, cfg, u)["q_all"]
    assert np.isfinite(got).all()

    last = np.zeros((2, N), bool)                    # an infinity in the last place, beside places past the row's end
    if D % 32:
        last[0, at.index(D - 1)] = True
        last[1, 0] = at[len(at) // 2] == D - 1
    want = oracle_unroll(cfg, pu.oracle_weights(cfg, w), None, u)["q_all"]
    check = lambda a, b, rows, what: np.testing.assert_allclose(np.moveaxis(a, 1, 2)[rows], np.moveaxis(b, 1, 2)[rows], atol=TOL, rtol=0, err_msg=what)
    check(got, want, ~last if D < 8 else np.ones_like(last), "oracle")

    h = np.zeros((2, N, H), np.float32)
    steps = []
    for t in range(T + 1):
        step = pu.gpu_act(net, cfg, dict(obs=u["obs"][:, t], avail=u["avail"][:, t], h_in=h, reset=None,
                                         step_t=np.full(2, t, np.int32), epsilon=0.0, seed=1))
        steps.append(step["q"])
        h = step["h_out"]
    check(got, np.stack(steps, 1), np.ones_like(last) if D < 8 else ~last, "decision step")
    net.close()


@pytest.mark.parametrize("D", [13, 161, 300])
def test_a_unit_without_weights_stays_at_zero(D):
    """A first-layer row of zeros has x = 0, and so no gradient, whatever stands in the places past the row's end."""
    cfg = dict(wl.config(0), N=4, D=D, A=6, H=64, dtype="bf16", B=2, T=4)
    w = wl.make_weights(cfg, 0).copy()
    at = {k: (a, b, w[a:b].reshape(shp)) for k, (a, b, shp) in wl.weight_slices(*wl.dims(cfg)).items()}
    at["W1"][2][::3] = 0
    at["b1"][2][::3] = 0
    u = wl.make_unroll_inputs(cfg)
    u["obs"][:] = 1 + np.abs(u["obs"])
    net = binding.QNet(wl.dims(cfg), w, "bf16")
    g = bptt.gpu_grad(net, cfg, u, np.ones(u["actions"].shape, np.float32))
    a, b, _ = at["W1"]
    grad = g[a:b].reshape(64, -1)
    assert (grad[::3] == 0).all() and (grad[1::3] != 0).any()
    net.close()
