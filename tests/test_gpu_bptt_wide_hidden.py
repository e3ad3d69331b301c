"""Gradients of bf16 networks with 128 hidden units where the reverse recurrence and the GRU matrices' products have their
edges, against the oracle with the bars of the gradient tests: episodes' rows fewer than a step of 32 samples and not a divisor
of it, one slot, odd and even numbers of slots walked in one launch and in two, samples just past a chunk's end, a first layer
whose product stays on narrow loads, one action and the most of them."""
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


@pytest.mark.parametrize("B,T,N,D,A", [(1, 1, 1, 8, 5), (9, 1, 2, 12, 5), (5, 3, 2, 8, 7), (11, 2, 5, 24, 64), (40, 7, 3, 12, 9),
                                       (3, 16, 1, 8, 17), (2, 17, 3, 20, 16), (7, 18, 3, 9, 33), (2, 33, 16, 16, 48), (13, 19, 5, 28, 1),
                                       (32, 16, 4, 8, 6), (33, 16, 4, 8, 6), (650, 3, 5, 12, 6)])
def test_gradient_at_the_edges_of_the_wide_backward_pass(B, T, N, D, A):
    cfg = dict(wl.config(4), N=N, D=D, A=A, H=128, dtype="bf16", B=B, T=T)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    # one sign: the sums grow with the samples as the oracle's ambiguity budget does
    g = np.abs(np.random.default_rng([B, T, N]).normal(size=(B, T, N))).astype(np.float32)
    net = binding.QNet(wl.dims(cfg), w, "bf16")
    got = bptt.gpu_grad(net, cfg, u, g)
    bptt.compare(cfg, got, *bptt.oracle_grad(cfg, w, u, g))
    assert (bptt.gpu_grad(net, cfg, u, g) == got).all()
    net.close()


GUARD_BYTES = 32 << 20             # more than the partial sums of both GRU products, 64 chunks of 384 x 144 each, take


@pytest.mark.parametrize("B,T,N,D,A", [(197, 13, 1, 8, 5), (64, 10, 5, 12, 6), (270, 5, 3, 12, 6), (273, 15, 1, 8, 64), (4, 16, 41, 8, 5)])
def test_nothing_is_written_behind_the_workspace(B, T, N, D, A):
    """One launch and 2561 to 4096 samples, where the GRU products would take more chunks than the other products and the
    workspace's end is theirs; the last shape in two launches."""
    cfg = dict(wl.config(4), N=N, D=D, A=A, H=128, dtype="bf16", B=B, T=T)
    w = wl.make_weights(cfg, 0)
    u = wl.make_unroll_inputs(cfg, B=B, T=T)
    # one sign: the sums grow with the samples as the oracle's ambiguity budget does
    g = np.abs(np.random.default_rng([B, T, N]).normal(size=(B, T, N))).astype(np.float32)
    net = binding.QNet(wl.dims(cfg), w, "bf16")
    need = net.grad_workspace_bytes(B, T)
    block = torch.full((need + GUARD_BYTES,), 0xA5, dtype=torch.uint8, device="cuda")
    got = bptt.gpu_grad(net, cfg, u, g, workspace=block[:need])
    assert (block[need:] == 0xA5).all()
    bptt.compare(cfg, got, *bptt.oracle_grad(cfg, w, u, g))
    net.close()
