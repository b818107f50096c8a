"""FC layer, core and heads of few rows in one launch (k_tail.hip): the bits of the three launches, at the edges of
the row tiles and on both sides of the limits, plain and with a state table, for both cells and every type of
features, with states that have no bf16 terms, and with workgroups that never start.  Every case asserts which of the
two a step takes, by the launches that it records."""
import ctypes

import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

_STD = dict(obs=(3, 72, 128), encoder="conv", convs=[(32, 8, 4, 0), (64, 4, 2, 0), (128, 3, 2, 0)], fc=512, rnn=512,
            dtype="fp32", rnn_type="gru", heads=[7], p_done=0.2, steps=1, obs_sub=0.0, obs_mul=wl.OBS_MUL, meas_dim=0,
            meas_hidden=[], index=5, name="tail")
_RES = dict(_STD, encoder="resnet", stages=[16, 32, 32], blocks_per_stage=2, fc=256, rnn=256, dtype="bf16", heads=[15])
# network, rows that take one launch (the last one: the most that do so, or close to it), rows that take three.  narrow: up
# to 1024 rows by its tiles, but only where workgroups share a frame of the first launch (up to 128 rows, 257 to 384)
_FEW = [1, 2, 15, 16, 17, 31]
NETS = {
    "gru": (_STD, _FEW + [33, 63, 64], [65]),
    "lstm": (dict(_STD, rnn_type="lstm"), _FEW + [33, 63, 64], [65]),
    "bf16": (dict(_STD, dtype="bf16"), _FEW + [33, 63, 64], [65]),
    "bf16-lstm": (dict(_STD, dtype="bf16", rnn_type="lstm", rnn=256, heads=[3, 3, 2, 2, 2, 8, 21]), _FEW + [111, 112], [113, 127]),
    "resnet": (_RES, _FEW + [127, 128], [129]),
    "resnet-lstm": (dict(_RES, rnn_type="lstm", heads=[30, 33]), _FEW + [127, 128], [129]),
    "heads": (dict(_STD, heads=[3, 3, 2, 2, 2, 8, 21]), _FEW + [63, 64], [65]),
    "narrow": (dict(_STD, fc=32, rnn=32, heads=[17, 5]), _FEW + [128, 257, 384], [129, 256, 385]),
    "wide": (dict(_STD, fc=480, rnn=1024), _FEW + [32], [33]),
}


def _policy(monkeypatch, net, max_batch, w, **env):
    for k, v in env.items():
        monkeypatch.setenv(k, str(v))
    pol = binding.Policy(net, w, max_batch=max_batch)
    for k in env:
        monkeypatch.delenv(k)
    return pol


def _inputs(torch, net, B, odd=False):
    x = dict(obs=wl.observations(net, 0, B), h=wl.initial_state(net, B), done=wl.done_mask(net, 0, B))
    if odd and B > 12:
        x["h"][3, 5], x["h"][7, 0], x["h"][11, 31] = np.inf, np.nan, 3.39e38
        x["h"][9].view(np.uint32)[2] = 0xFFFFFFFF
    return {k: torch.from_numpy(v).cuda() for k, v in x.items()}


def _step(torch, pol, x, B):
    out = pol.step(x["obs"][:B], x["h"][:B], x["done"][:B], 7, 11)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def _indexed(torch, pol, x, B, ids, n_env):
    table = torch.full((n_env, pol.H), 3.0, device="cuda")
    ok = (ids >= 0) & (ids < n_env)
    table[ids[ok].long()] = x["h"][:B][ok]
    out = pol.step_indexed(x["obs"][:B], table, ids, x["done"][:B], 7, 11)
    torch.cuda.synchronize()
    return dict({k: v.cpu().numpy() for k, v in out.items()}, table=table.cpu().numpy())


def _same(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=a[k].dtype.kind == "f"), (what, k)


def _launches(torch, pol, x, B):
    """Launches of a plain step, recorded."""
    out = pol.alloc_outputs(B)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        pol.step(x["obs"][:B], x["h"][:B], x["done"][:B], 7, 11, out=out, stream=torch.cuda.current_stream())
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("name", NETS)
def test_bits_of_the_three_launches(torch_cuda, monkeypatch, name):
    torch = torch_cuda
    net, in_one, in_three = NETS[name]
    B, most = max(in_one + in_three), in_one[-1]
    w = wl.weights(net)
    one, three = _policy(monkeypatch, net, B, w), _policy(monkeypatch, net, B, w, SF_NO_TAIL=1)
    x = _inputs(torch, net, B)
    odd = _inputs(torch, net, B, odd=True)
    for n in sorted(in_one + in_three):
        print(name, n, flush=True)
        _same(_step(torch, one, x, n), _step(torch, three, x, n), n)
        assert _launches(torch, three, x, n) - _launches(torch, one, x, n) == (2 if n in in_one else 0), n
    _same(_step(torch, one, odd, most), _step(torch, three, odd, most), "states without terms")
    ids = torch.from_numpy(np.random.default_rng(3).permutation(2 * B)[:B].astype(np.int32)).cuda()
    ids[0], ids[most - 2] = -1, 2 * B
    for n in (1, 17, most):
        _same(_indexed(torch, one, x, n, ids[:n], 2 * B), _indexed(torch, three, x, n, ids[:n], 2 * B), ("table", n))
    _same(_indexed(torch, one, odd, most, ids[:most], 2 * B), _indexed(torch, three, odd, most, ids[:most], 2 * B), "table, states without terms")
    one.close()
    three.close()


@pytest.mark.parametrize("name,B", [("gru", 33), ("lstm", 50), ("bf16", 60), ("resnet-lstm", 100)])
def test_workgroups_that_never_start(torch_cuda, monkeypatch, name, B):
    """The others take over the roles of the first workgroups, down to one that computes everything; the heads have
    to run themselves, so that a larger number is taken for that of the FC and cell tiles.  Plain, and with a state
    table, whose writers take over, too."""
    torch = torch_cuda
    net = NETS[name][0]
    w = wl.weights(net)
    x = _inputs(torch, net, B)
    ids = torch.from_numpy(np.random.default_rng(4).permutation(2 * B)[:B].astype(np.int32)).cuda()
    ids[B - 5] = 2 * B
    pol = _policy(monkeypatch, net, B, w)
    want, want_table = _step(torch, pol, x, B), _indexed(torch, pol, x, B, ids, 2 * B)
    n = _launches(torch, pol, x, B)
    pol.close()
    pol = _policy(monkeypatch, net, B, w, SF_NO_TAIL=1)
    assert _launches(torch, pol, x, B) == n + 2
    pol.close()
    tiles, fc, cell = (B + 15) // 16, net["fc"] // 16, net["rnn"] // 8
    for skip in (1, tiles * fc - 1, tiles * fc + 3, tiles * (fc + cell) - 1, tiles * (fc + cell + 1), 100000):
        print(name, "without the first", skip, flush=True)
        pol = _policy(monkeypatch, net, B, w, SF_TAIL_SKIP=skip)
        for _ in range(2):
            _same(_step(torch, pol, x, B), want, skip)
            _same(_indexed(torch, pol, x, B, ids, 2 * B), want_table, (skip, "table"))
        pol.close()


@pytest.mark.parametrize("name", ["gru", "lstm", "bf16", "resnet-lstm", "narrow"])
def test_two_rows_of_one_environment(torch_cuda, monkeypatch, name):
    """Rows of the batch that name the same environment, in one row tile and in several: each is computed from the
    environment's old state, and the table receives the state of one of them, the last; recorded, too."""
    torch = torch_cuda
    net, in_one, _ = NETS[name]
    B = min(in_one[-1], 100) - 3
    w = wl.weights(net)
    pol, three = _policy(monkeypatch, net, B, w), _policy(monkeypatch, net, B, w, SF_NO_TAIL=1)
    x = _inputs(torch, net, B)
    n_env = 2 * B
    ids = np.random.default_rng(5).permutation(n_env)[:B].astype(np.int32)
    ids[40], ids[7], ids[20], ids[B - 1], ids[B - 2], ids[17] = ids[3], ids[5], ids[1], ids[1], ids[0], n_env
    last = {int(e): b for b, e in enumerate(ids) if e < n_env}
    ids = torch.from_numpy(ids).cuda()
    old = 0.1 * torch.randn(n_env, pol.H, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    h = torch.where((ids < n_env)[:, None], old[ids.clamp(max=n_env - 1).long()], torch.zeros((), device="cuda"))
    state = pol.step(x["obs"], h, x["done"], 7, 11)["h_out"]
    new = old.clone()
    for e, b in last.items():
        new[e] = state[b]
    table = old.clone()
    want = three.step_indexed(x["obs"], table, ids, x["done"], 7, 11)
    assert _launches(torch, three, x, B) - _launches(torch, pol, x, B) == 2

    def check(got):
        torch.cuda.synchronize()
        for k in got:
            assert torch.equal(got[k], want[k]), k
        assert torch.equal(table, new)

    for _ in range(10):
        table.copy_(old)
        check(pol.step_indexed(x["obs"], table, ids, x["done"], 7, 11))
    out = pol.alloc_outputs(B)
    del out["h_out"]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pol.step_indexed(x["obs"], table, ids, x["done"], 7, 11, out=out, stream=torch.cuda.current_stream())
    for _ in range(4):  # with eager work and synchronisations between the replays
        table.copy_(old)
        for v in out.values():
            v.zero_()
        torch.cuda.synchronize()
        graph.replay()
        check(out)
    pol.close()
    three.close()
