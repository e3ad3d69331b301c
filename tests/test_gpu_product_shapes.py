"""Gradients whose weight products sit at the edges of the product kernels' tiles (128 x 176 and 128 x 336, 256 x 80 and
256 x 144, 384 x 144), against the oracle with the bars of the gradient tests."""
import numpy as np
import pytest
import torch

from oracle import mixer_oracle as mxo
from paper_2205_05248_amd import binding, workloads as wl
import test_gpu_bptt as bptt
import test_gpu_mixer as mixer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


# D + N: one column short of, exactly and one past the narrower first-layer tile; with bf16 weights an observation size that
# is a whole number of 16-byte pieces and one that is not; 128 units beside them
@pytest.mark.parametrize("N,D,H,dtype", [(15, 160, 64, "fp32"), (16, 160, 64, "fp32"), (17, 160, 64, "fp32"),
                                         (16, 160, 64, "bf16"), (17, 160, 64, "bf16"), (16, 159, 64, "bf16"), (20, 157, 64, "bf16"),
                                         (16, 160, 128, "bf16"), (17, 160, 128, "bf16")])
def test_first_layer_gradient_around_a_tile(N, D, H, dtype):
    cfg = dict(wl.config(0), N=N, D=D, H=H, A=10, dtype=dtype, B=3, T=18)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=3, T=18)
    g = np.random.default_rng(N + D).standard_normal(u["actions"].shape).astype(np.float32)
    net = binding.QNet(wl.dims(cfg), w, dtype)
    bptt.compare(cfg, bptt.gpu_grad(net, cfg, u, g), *bptt.oracle_grad(cfg, w, u, g))
    net.close()


def compare_mixer_gradient(dims, dtype, B, T):
    """One switch (the sign of a generated weight, an offset unit) within the forward error of zero may be worth more than the
    cap that the comparison sets on the oracle's ambiguity budget, where there are few transitions.  The inputs are the first, of
    twenty, whose budget is within the cap; that is decided by the oracle alone."""
    N, M, S = dims
    cfg = dict(wl.config(0), N=N, S=S, B=B, T=T)
    m = wl.make_mixer_inputs(cfg)
    e = np.abs(np.random.default_rng([12, N, S]).normal(size=(B, T))).astype(np.float32) * m["filled"]
    for seed in range(20):
        w = wl.pack_mixer(dims, {k: np.random.default_rng([seed, i]).uniform(-1, 1, shp) / np.sqrt(max(shp[-1], 1) if len(shp) == 2 else 4)
                                 for i, (k, (_, _, shp)) in enumerate(wl.mixer_slices(*dims).items())})
        _, want, budget = mxo.grad(dims, mixer.oracle_mixer_weights(dims, w, dtype), m["state"], m["q_taken"].astype(np.float64),
                                   e.astype(np.float64), switch_band=mixer.SWITCH_BAND[dtype], inputs_as_bf16=dtype == "bf16")
        if all(budget[a:b].max() <= mixer.BUDGET_CAP * np.abs(want[a:b]).max() for a, b, _ in wl.mixer_slices(*dims).values()):
            break
    else:
        pytest.fail("no inputs within the budget's cap")
    mixer._compare_mixer_gradient("N%d M%d S%d" % dims, dims, w, dtype, m, e)


# agents x hidden units: the rows of the largest product; state sizes: its columns, whole slices and one past them
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("N,M,S", [(8, 16, 64), (9, 16, 64), (9, 16, 65), (16, 16, 79), (16, 16, 80), (17, 16, 128), (24, 16, 129),
                                   (25, 16, 48), (2, 64, 176), (3, 64, 177)])
def test_mixer_gradient_around_a_tile(N, M, S, dtype):
    compare_mixer_gradient((N, M, S), dtype, 5, 31)


# Lists of products: rows of one class only if cut into one slice more (528, 784), even slices of unequal blocks (800, 1024); more
# than sixteen tall products, in two launches and in three of unequal size; seventeen flat ones.  Several chunks of transitions each.
@pytest.mark.parametrize("N,M,S,dtype", [(33, 16, 129, "fp32"), (49, 16, 100, "bf16"), (25, 32, 128, "bf16"), (32, 32, 132, "bf16"),
                                         (51, 32, 400, "fp32"), (32, 64, 300, "bf16"), (57, 64, 420, "bf16"), (8, 16, 1000, "bf16")])
def test_mixer_gradient_of_many_products(N, M, S, dtype):
    compare_mixer_gradient((N, M, S), dtype, 9, 57)
