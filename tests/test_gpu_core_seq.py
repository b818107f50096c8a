"""The recurrent core over all time steps in one launch (k_core_seq.hip): every number of K steps per wave,
one and two row tiles per workgroup, ragged rows, more workgroups than the chip has CUs, states that are
not finite, and the pass that gives up its exchange and is computed again without one."""
import ctypes as C

import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

BASE = dict(obs=(3, 36, 64), convs=[(16, 8, 4, 0), (32, 4, 2, 0)], p_done=0.2)
# name, T, N, network: features + state -> K steps per wave (32 numbers each, eight waves)
CASES = {
    "gru-1-1": (5, 20, dict(fc=96, rnn=32)),
    "gru-1-1-two-tiles": (5, 500, dict(fc=128, rnn=128)),
    "lstm-2-1": (6, 7, dict(fc=288, rnn=64, rnn_type="lstm")),
    "gru-2-2-two-tiles": (6, 116, dict(fc=512, rnn=512)),
    "lstm-2-2": (5, 12, dict(fc=512, rnn=288, rnn_type="lstm")),
    "gru-3-2-two-rounds": (6, 120, dict(fc=512, rnn=512, meas_dim=23, meas_hidden=[64, 128])),
    "bf16-gru-2-2-two-tiles": (6, 124, dict(fc=512, rnn=512, dtype="bf16")),
    "one-launch-per-step": (3, 20, dict(fc=96, rnn=32)),
    "bf16-lstm-1-1": (5, 24, dict(fc=128, rnn=96, rnn_type="lstm", dtype="bf16")),
    "lstm-2-2-learner": (32, 64, dict(fc=512, rnn=512, rnn_type="lstm")),
}


def _pass(torch, net, w, T, N, env, monkeypatch, h0=None, ends=()):
    with monkeypatch.context() as m:
        for k, v in env.items():
            m.setenv(k, v)
        pol = binding.Policy(net, w, max_batch=T * N)
    obs, h, done, meas = wl.trajectory_inputs(net, T, N)
    h = h if h0 is None else h0
    for at in ends:
        done[at] = 1
    out = pol.unroll(*(torch.from_numpy(a).cuda() for a in (obs, h, done)),
                     meas=None if meas is None else torch.from_numpy(meas).cuda())
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    pol.close()
    return got, (obs, h, done, meas)


@pytest.mark.parametrize("name", CASES)
def test_one_launch_for_all_steps(torch_cuda, ref, monkeypatch, name):
    torch = torch_cuda
    T, N, kw = CASES[name]
    net = wl.network(0, **dict(BASE, name=name, **kw))
    w = wl.weights(net)
    got, (obs, h0, done, meas) = _pass(torch, net, w, T, N, {}, monkeypatch)
    rtol = parity.RTOL[net["dtype"]]
    sel = np.unique(np.array([0, N // 3, N - 1]))
    want = ref.policy_unroll(net, w, obs[:, sel], h0[sel], done[:, sel],
                             meas=None if meas is None else meas[:, sel])
    for k in ("h_seq", "logits", "value"):
        parity.assert_close(k, got[k][:, sel], want[k], rtol)
    # every element: a launch per step, and the pass that gives up; both add the same terms in other orders
    for env in ({"SF_NO_RNN_SEQ": "1"}, {"SF_CORE_SEQ_LIMIT": "-1"}):
        other, _ = _pass(torch, net, w, T, N, env, monkeypatch)
        for k in ("h_seq", "logits", "value"):
            parity.assert_close(k, got[k], other[k], rtol)


@pytest.mark.parametrize("kind,T,N,size", [("gru", 5, 24, (96, 64)), ("lstm", 5, 24, (96, 64)),
                                           ("gru", 6, 116, (512, 512)), ("lstm", 32, 64, (512, 512))])
def test_states_that_are_not_finite(torch_cuda, monkeypatch, kind, T, N, size):
    """A row that starts with an infinity, a NaN, the NaN that marks a state as still to come, or a number
    whose products overflow: the same kind of number everywhere as with a launch per step, also behind the
    end of its episode, and every other row, of the same row tile too, has the bits that it has without such
    neighbours."""
    torch = torch_cuda
    net = wl.network(0, **dict(BASE, name="odd_" + kind, fc=size[0], rnn=size[1], rnn_type=kind, p_done=0.0))
    w = wl.weights(net)
    w["rnn_w_hh"] = w["rnn_w_hh"].copy()
    w["rnn_w_hh"][:, 0] = np.where(w["rnn_w_hh"][:, 0] > 0, 4.0, -4.0)
    clean = wl.trajectory_inputs(net, T, N)[1]
    h0 = clean.copy()
    h0[3, 5] = np.inf
    h0[9, 60] = np.nan
    h0.view(np.uint32)[17, :] = 0xFFFFFFFF
    h0[20, 0] = 3e38
    ends = [(2, 9), (T - 1, 17)]  # (step, row): a new episode
    got, _ = _pass(torch, net, w, T, N, {}, monkeypatch, h0, ends)
    other, _ = _pass(torch, net, w, T, N, {"SF_NO_RNN_SEQ": "1"}, monkeypatch, h0, ends)
    without, _ = _pass(torch, net, w, T, N, {}, monkeypatch, clean, ends)
    rows = [r for r in range(N) if r not in (3, 9, 17, 20)]
    for k in got:
        assert np.array_equal(np.isnan(got[k]), np.isnan(other[k])), k
        parity.assert_close(k, np.nan_to_num(got[k]), np.nan_to_num(other[k]), 1e-4)
        assert np.array_equal(got[k][:, rows], without[k][:, rows]), k
    assert np.isfinite(without["h_seq"]).all()
    for t, r in ends:
        assert np.isnan(got["h_seq"][t - 1, r]).any() and np.isfinite(got["h_seq"][t:, r]).all()
        assert np.array_equal(got["h_seq"][t:, r], without["h_seq"][t:, r])


def _same_as_single_steps(pol, args, stream=None):
    """Whether a pass has the bits of passes of one step each (a launch per step), by step."""
    obs, h0, done = args
    got = {k: v.cpu().numpy() for k, v in pol.unroll(obs, h0, done, stream=stream).items()}
    same, h = [], h0
    for t in range(obs.shape[0]):
        out = pol.unroll(obs[t:t + 1], h, done[t:t + 1])
        same.append(all(np.array_equal(out[k][0].cpu().numpy(), got[k][t]) for k in got))
        h = out["h_seq"][0].clone()
    return same


def test_compute_units_that_a_row_tile_needs(torch_cuda, monkeypatch):
    """The workgroups of a row tile wait for one another: on fewer compute units than they are (SF_CUS), and
    where the pass would take several rounds of workgroups, a launch per step."""
    torch = torch_cuda
    net = wl.network(0, **dict(BASE, name="few_units", fc=512, rnn=512))
    w = wl.weights(net)
    T = 6
    for N, cus, one_launch in ((16, 0, True), (16, 64, True), (16, 63, False), (64, 128, True), (64, 127, False)):
        with monkeypatch.context() as m:
            if cus:
                m.setenv("SF_CUS", str(cus))
            pol = binding.Policy(net, w, max_batch=T * N)
        same = _same_as_single_steps(pol, [torch.from_numpy(a).cuda() for a in wl.trajectory_inputs(net, T, N)[:3]])
        pol.close()
        assert all(same) != one_launch, (N, cus, same)


@pytest.mark.parametrize("H,N,shortest", [(32, 16, 4), (32, 17, 5), (256, 16, 4), (256, 40, 5), (512, 16, 4), (512, 17, 6)])
def test_short_passes(torch_cuda, H, N, shortest):
    """Passes of fewer steps than pay for the one launch take a launch per step."""
    torch = torch_cuda
    net = wl.network(0, **dict(BASE, name="short", fc=H, rnn=H))
    pol = binding.Policy(net, wl.weights(net), max_batch=shortest * N)
    for T in (shortest - 1, shortest):
        same = _same_as_single_steps(pol, [torch.from_numpy(a).cuda() for a in wl.trajectory_inputs(net, T, N)[:3]])
        assert all(same) == (T < shortest), (T, same)
    pol.close()


def test_stream_with_a_mask(torch_cuda):
    """The same for a stream that may not use all compute units: 128 rows of 512 units take 256 of them."""
    torch = torch_cuda
    units = torch.cuda.get_device_properties(0).multi_processor_count
    if units != 256:
        pytest.skip("sizes are those of 256 compute units")
    hip = C.CDLL("libamdhip64.so")
    mask, raw = (C.c_uint32 * 8)(*[0xFFFFFF00] + [0xFFFFFFFF] * 7), C.c_void_p()
    if hip.hipExtStreamCreateWithCUMask(C.byref(raw), C.c_uint32(8), mask) != 0:
        pytest.skip("no streams with a mask here")
    net = wl.network(0, **dict(BASE, name="masked", fc=512, rnn=512))
    T, N = 6, 128
    pol = binding.Policy(net, wl.weights(net), max_batch=T * N)
    args = [torch.from_numpy(a).cuda() for a in wl.trajectory_inputs(net, T, N)[:3]]
    torch.cuda.synchronize()
    assert not all(_same_as_single_steps(pol, args))
    stream = torch.cuda.ExternalStream(raw.value)
    with torch.cuda.stream(stream):
        assert all(_same_as_single_steps(pol, args, stream))
    stream.synchronize()
    pol.close()
    assert hip.hipStreamDestroy(raw) == 0


def test_two_passes_at_once(torch_cuda, monkeypatch):
    """Two handles on two streams, each with as many workgroups as the chip has compute units: the bits of a
    pass alone."""
    torch = torch_cuda
    T, N = 32, 64
    pair = []
    for kind in ("gru", "lstm"):
        net = wl.network(0, **dict(BASE, name="pair_" + kind, fc=512, rnn=512, rnn_type=kind))
        pol = binding.Policy(net, wl.weights(net), max_batch=T * N)
        args = tuple(torch.from_numpy(a).cuda() for a in wl.trajectory_inputs(net, T, N)[:3])
        alone = {k: v.clone() for k, v in pol.unroll(*args).items()}
        out = {k: torch.zeros_like(v) for k, v in alone.items()}
        pair.append((pol, args, alone, out, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(4):
        for pol, args, _, out, stream in pair:
            pol.unroll(*args, out=out, stream=stream)
    torch.cuda.synchronize()
    for pol, _, alone, out, _ in pair:
        for k in alone:
            assert torch.equal(alone[k], out[k]), k
        pol.close()
