"""GPU parity of fp32 networks with 128 hidden units, whose unroll runs the recurrence on tiles of 16 rows that share
records of 32 rows with a neighbour: row counts around the tile and the record, the shortest episodes and odd and even
numbers of slots, every number of action blocks, all three forms of the TD step."""
import numpy as np
import pytest
import torch

from paper_2205_05248_amd import binding, workloads as wl
import parity_util as pu
from test_gpu_parity import compare_double, make_net, oracle_unroll, run_double

pytestmark = pytest.mark.gpu
TOL = pu.TOL["fp32"]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


SHAPES = [
    # B, T, N, D, A
    (1, 1, 1, 1, 1),         # one row, two slots, fewer actions than a lane holds; observations of less than eight values
    (1, 2, 16, 8, 3),        # one whole tile, half a record; the fewest observations the weight-stationary projection takes
    (1, 3, 17, 33, 4),       # one row past a tile; observations one past a k-step
    (2, 4, 16, 64, 16),      # one whole record
    (3, 5, 11, 55, 17),      # one row past a record; a second action block of one action
    (5, 6, 13, 97, 48),      # an odd number of tiles
    (7, 25, 30, 161, 64),    # the most actions, 210 rows
    (2, 9, 3, 255, 5),       # eight k-steps, one observation short of whole
    (9, 31, 5, 257, 40),     # ten k-steps with one empty
    (3, 40, 64, 320, 9),     # the widest; more items than workgroups
    (4, 7, 5, 321, 9),       # wider: the streaming projection
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d_T%d_N%d_D%d_A%d" % s)
def test_unroll_of_wide_fp32_networks(shape):
    B, T, N, D, A = shape
    cfg = dict(wl.config(0), B=B, T=T, N=N, D=D, A=A, H=128, dtype="fp32")
    net, w = make_net(cfg)
    target, w_tg = make_net(cfg, 1)
    u = wl.make_unroll_inputs(cfg)
    got = pu.gpu_unroll(net, target, cfg, u)
    pu.compare_unroll(got, oracle_unroll(cfg, w, w_tg, u), TOL)
    # one network, no Q values kept: the same online half bit for bit
    one = pu.gpu_unroll(net, None, cfg, u, want_q_all=False)
    np.testing.assert_array_equal(one["q_taken"], got["q_taken"])
    pu.compare_unroll(one, dict(oracle_unroll(cfg, w, None, u), q_all=None), TOL)
    # the double estimator, packed and from a pool
    keys = ["obs", "avail", "actions", "reward", "terminated", "filled"]
    d = pu.to_dev(u, keys)
    double = run_double(net, target, cfg, u, d)
    compare_double(cfg, u, double, w, w_tg, TOL)
    pick = np.random.default_rng(B).integers(0, B, B + 2).astype(np.int32)
    pooled = run_double(net, target, cfg, u, d, index=pick)
    for k in ("q_taken", "next_max", "td_target", "next_action", "q_all"):
        np.testing.assert_array_equal(pooled[k], double[k][pick])
    net.close(); target.close()
