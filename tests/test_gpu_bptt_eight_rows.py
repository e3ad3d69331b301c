"""Gradients of networks with 64 hidden units around a tile of eight rows, which the reverse recurrence takes where a batch leaves
compute units free: rows one short of, exactly and one past whole tiles, odd and even numbers of slots, every number of blocks
that the adjoint of Q has, against the oracle with the bars of the gradient tests."""
import numpy as np
import pytest
import torch

from paper_2205_05248_amd import binding, workloads as wl
import test_gpu_bptt as bptt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("B,T,N,A", [(7, 5, 1, 5), (8, 6, 1, 17), (9, 5, 1, 33), (5, 7, 3, 64), (4, 17, 4, 16), (3, 16, 11, 40)])
def test_gradient_around_a_tile_of_eight_rows(dtype, B, T, N, A):
    cfg = dict(wl.config(0), N=N, A=A, dtype=dtype, B=B, T=T)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    # one sign: the sums grow with the samples as the oracle's ambiguity budget does
    g = np.abs(np.random.default_rng([B, T, A]).normal(size=(B, T, N))).astype(np.float32)
    net = binding.QNet(wl.dims(cfg), w, dtype)
    got = bptt.gpu_grad(net, cfg, u, g)
    bptt.compare(cfg, got, *bptt.oracle_grad(cfg, w, u, g))
    assert (bptt.gpu_grad(net, cfg, u, g) == got).all()
    net.close()


def test_no_row_past_the_last_one_reaches_the_adjoints_of_a_large_fp32_batch():
    """Adjoints of more than 2^31 bytes and a last tile that is not full.  The upstream gradient is non-zero for four episodes, of
    which two have their adjoints around 2^31 bytes, so the oracle has to walk just those (the sum is linear in it)."""
    B, T, N = 409, 1100, 5
    cfg = dict(wl.config(0), N=N, D=8, A=5, dtype="fp32", B=B, T=T)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    u["filled"][:] = 1
    around = (1 << 31) // (4 * 64 * 4 * N * T)
    live = [0, around, around + 1, B - 1]
    g = np.zeros((B, T, N), np.float32)
    # one sign: the sums grow with the samples as the oracle's ambiguity budget does
    g[live] = np.abs(np.random.default_rng([B, T, N]).normal(size=(len(live), T, N)))
    net = binding.QNet(wl.dims(cfg), w, "fp32")
    got = bptt.gpu_grad(net, cfg, u, g)
    sub = {k: np.ascontiguousarray(u[k][live]) for k in ("obs", "actions", "filled")}
    bptt.compare(cfg, got, *bptt.oracle_grad(cfg, w, sub, g[live]))
    net.close()
