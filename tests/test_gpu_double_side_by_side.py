"""The double-estimator call whose two networks run side by side: the same bits as the two launches one after the other,
which is what a captured call runs, over row counts around a tile (16) and a record (32), the fewest and most actions
and all networks of the fused kernels; which of the two ways a call goes, by the room that one of them takes; and calls of one
handle on two streams at once."""
import numpy as np
import pytest
import torch

from paper_2205_05248_amd import binding, workloads as wl
import parity_util as pu
from test_gpu_parity import compare_double, make_net

pytestmark = pytest.mark.gpu
KEYS = ["obs", "avail", "actions", "reward", "terminated", "filled"]
NAMES = ("q_taken", "next_max", "td_target", "next_action", "q_all")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    binding.load()
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


def blank(cfg, B):
    N, _, A, _ = wl.dims(cfg)
    T = cfg["T"]
    out = {k: torch.full((B, T, N), float("nan"), device="cuda") for k in NAMES[:3]}
    out["next_action"] = torch.full((B, T, N), -9, dtype=torch.int32, device="cuda")
    out["q_all"] = torch.full((B, T + 1, N, A), float("nan"), device="cuda")
    return out


def call(net, target, d, gamma, out, index=None):
    net.unroll_td_double(target, *(d[k] for k in KEYS), gamma, *(out[k] for k in NAMES), index)


SHAPES = [
    # B, T, N, D, A, H, dtype
    (1, 1, 1, 9, 1, 64, "fp32"),
    (1, 2, 16, 30, 5, 64, "bf16"),
    (3, 3, 11, 20, 16, 128, "bf16"),
    (17, 7, 2, 33, 17, 64, "fp32"),
    (13, 20, 5, 55, 64, 128, "bf16"),
    (150, 3, 20, 31, 6, 64, "fp32"),     # 188 tiles: twice the chip either way, one after the other
    (290, 2, 16, 31, 6, 64, "bf16"),     # 290 tiles: side by side again
    (2, 4, 3, 1000, 7, 64, "fp32"),      # too wide for the fused kernels: one after the other either way
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d_T%d_N%d_D%d_A%d_H%d_%s" % s)
def test_side_by_side_gives_the_bits_of_one_after_the_other(shape):
    B, T, N, D, A, H, dtype = shape
    cfg = dict(wl.config(0), B=B, T=T, N=N, D=D, A=A, H=H, dtype=dtype)
    net, w = make_net(cfg)
    target, w_tg = make_net(cfg, 1)
    binding.marl_qnet_reserve_unroll(net.handle, B, T)
    binding.marl_qnet_reserve_unroll(target.handle, B, T)
    u = wl.make_unroll_inputs(cfg)
    u["avail"][0, 1, 0, :] = 0
    d = pu.to_dev(u, KEYS)
    index = torch.from_numpy(np.random.default_rng(B).integers(0, B, B).astype(np.int32)).cuda()
    for pick in (None, index):
        eager, replayed = blank(cfg, B), blank(cfg, B)
        call(net, target, d, u["gamma"], eager, pick)
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
            call(net, target, d, u["gamma"], replayed, pick)
        torch.cuda.synchronize()
        for _ in range(2):
            for k in NAMES:
                replayed[k].fill_(-5)
            graph.replay()
            again = blank(cfg, B)
            call(net, target, d, u["gamma"], again, pick)
            torch.cuda.synchronize()
            for k in NAMES:
                assert torch.equal(eager[k], replayed[k]) and torch.equal(eager[k], again[k]), k
        if pick is None:
            compare_double(cfg, u, {k: v.cpu().numpy() for k, v in eager.items()}, w, w_tg, pu.TOL[dtype])
    net.close(); target.close()


def test_room_grows_while_an_earlier_call_is_in_flight():
    """A small batch on one stream, then one that needs more room on another, with nothing waited for in between."""
    cfg = dict(wl.config(1), T=60)
    N, D, A, H = wl.dims(cfg)
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    sizes = (6, 40)
    assert all(2 * ((B * N + 15) // 16) <= 256 for B in sizes)              # side by side, either one
    (first, _), (target, _) = make_net(cfg), make_net(cfg, 1)
    batches = []
    for s, B in enumerate(sizes):
        u = wl.make_unroll_inputs(cfg, B=B, T=60, stream=s)
        d, want = pu.to_dev(u, KEYS), blank(cfg, B)
        call(first, target, d, u["gamma"], want)
        batches.append((u, d, want))
    torch.cuda.synchronize()
    for _ in range(3):
        net, _ = make_net(cfg)                                              # room for nothing yet
        got = [blank(cfg, B) for B in sizes] + [blank(cfg, sizes[0])]
        torch.cuda.synchronize()
        for turn, out in enumerate(got):
            u, d, _ = batches[turn % 2]
            with torch.cuda.stream(streams[turn % 2]):
                call(net, target, d, u["gamma"], out)
        torch.cuda.synchronize()
        for turn, out in enumerate(got):
            for k in NAMES:
                assert torch.equal(out[k], batches[turn % 2][2][k]), (turn, k)
        net.close()
    first.close(); target.close()


def test_one_handle_on_two_streams():
    """Batches of different sizes enqueued in turn on two streams with nothing waited for in between."""
    cfg = dict(wl.config(1), T=30)
    net, _ = make_net(cfg)
    target, _ = make_net(cfg, 1)
    batches = []
    for s, B in enumerate((40, 9)):
        u = wl.make_unroll_inputs(cfg, B=B, T=30, stream=s)
        d, want, got = pu.to_dev(u, KEYS), blank(cfg, B), [blank(cfg, B) for _ in range(4)]
        call(net, target, d, u["gamma"], want)
        batches.append((u, d, want, got, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for turn in range(4):
        for u, d, want, got, stream in batches:
            with torch.cuda.stream(stream):
                call(net, target, d, u["gamma"], got[turn])
    torch.cuda.synchronize()
    for u, d, want, got, stream in batches:
        for out in got:
            for k in NAMES:
                assert torch.equal(out[k], want[k]), k
    net.close(); target.close()


# B, T, N, D, A, H, dtype, whether its networks run side by side
ROOMS = [(64, 200, 32, 30, 40, 128, "bf16", True),        # 128 tiles of 16 rows: both networks fill the chip once
         (100, 200, 20, 30, 40, 64, "bf16", True),        # 125
         (100, 200, 20, 30, 40, 64, "fp32", True),
         (128, 200, 20, 30, 40, 64, "bf16", False)]       # 160: twice the chip either way


@pytest.mark.parametrize("shape", ROOMS, ids=lambda s: "B%d_T%d_N%d_D%d_A%d_H%d_%s_%s" % s)
def test_room_is_made_by_the_call_that_needs_it_and_given_back(shape):
    """The target's Q values, over 60 MB here, have their room made in the way through a call that runs both networks side by side,
    and nowhere else: not by reserving, by the plain unroll, by a captured call, or where the networks run one after the other."""
    B, T, N, D, A, H, dtype, side_by_side = shape
    cfg = dict(wl.config(0), B=B, T=T, N=N, D=D, A=A, H=H, dtype=dtype)
    u = wl.make_unroll_inputs(cfg)
    d, out = pu.to_dev(u, KEYS), blank(cfg, B)
    need = 4 * B * (T + 1) * N * A
    assert 60 << 20 <= need <= 256 << 20
    plain = lambda: net.unroll_td(target, *(d[k] for k in KEYS), u["gamma"], *(out[k] for k in NAMES[:3]), out["q_all"])
    stream = torch.cuda.Stream()

    def captured():
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            call(net, target, d, u["gamma"], out)

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    net, _ = make_net(cfg)
    target, _ = make_net(cfg, 1)
    plain(); captured()                                    # whatever first launches and a first capture take
    before = free()
    for handle in (net.handle, target.handle):
        binding.marl_qnet_reserve_unroll(handle, B, T)
    plain(); captured()
    assert before - free() < need // 2
    for _ in range(2):
        call(net, target, d, u["gamma"], out)
        assert (need // 2 < before - free() < 2 * need) if side_by_side else before - free() < need // 2
    net.close(); target.close()
    assert before - free() < need // 2
