"""The heads on split operands (heads_split_kernel): output counts at the edges of its column tiles
and of its range, rows at the edges of its row tile, waves without a K step, many and single-category
heads, and states that hold an infinity or a NaN."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

_BASE = dict(obs=(3, 36, 64), encoder="conv", convs=[(16, 8, 4, 0), (32, 4, 2, 0)], dtype="fp32", p_done=0.2, steps=1,
             obs_sub=0.0, obs_mul=wl.OBS_MUL, meas_dim=0, meas_hidden=[], rnn_type="gru", index=5, name="heads")
CASES = [(dict(heads=[15], rnn=64), 16), (dict(heads=[16], rnn=64), 17), (dict(heads=[31], rnn=32), 1),
         (dict(heads=[40, 8], rnn=96), 33), (dict(heads=[63], rnn=288), 40), (dict(heads=[64], rnn=64), 20),
         (dict(heads=[1] * 15 + [5], rnn=64), 19), (dict(heads=[4, 4, 4, 5], rnn=64, rnn_type="lstm"), 50),
         (dict(heads=[3, 3, 2, 2, 2, 8, 21], rnn=128, dtype="bf16"), 37)]


@pytest.mark.parametrize("kw,B", CASES, ids=["%s-%d-%d" % ("+".join(map(str, k["heads"])), k["rnn"], b) for k, b in CASES])
def test_heads(torch_cuda, ref, kw, B):
    torch = torch_cuda
    net = dict(_BASE, fc=64, **kw)
    w = wl.weights(net)
    pol = binding.Policy(net, w, max_batch=B)
    d = pol.device
    obs, state, done = wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B)
    args = [torch.from_numpy(a).to(d) for a in (obs, state, done)]
    g = {k: v.cpu().numpy() for k, v in pol.step(*args, 7, 11).items()}
    torch.cuda.synchronize()
    parity.check_against_oracle(net, g, ref.policy_step(net, w, obs, state, done, 7, 11), ref, 7, 11)
    pol.close()


def test_rows_without_terms(torch_cuda):
    """A row whose state holds a NaN has NaN logits; one with a number that rounds up to an infinity in bf16,
    in one unit, has the plain sums; the other rows keep their bits."""
    torch = torch_cuda
    net = dict(_BASE, fc=64, rnn=64, heads=[7])
    w = wl.weights(net)
    # unit 9 keeps a large state: its z gate opens with it, and every r gate (no 0 * infinity in an n gate)
    H, unit, most = 64, 9, np.finfo(np.float32).max
    w["rnn_w_hh"][:H, unit] = np.abs(w["rnn_w_hh"][:H, unit])
    w["rnn_w_hh"][H + unit, unit] = np.abs(w["rnn_w_hh"][H + unit, unit])
    pol = binding.Policy(net, w, max_batch=20)
    d = pol.device
    obs, state, done = wl.observations(net, 0, 20), wl.initial_state(net, 20), np.zeros(20, np.uint8)
    run = lambda s: {k: v.cpu().numpy() for k, v in pol.step(torch.from_numpy(obs).to(d), torch.from_numpy(s).to(d),
                                                             torch.from_numpy(done).to(d), 7, 11).items()}
    clean = run(state)
    odd = state.copy()
    odd[3, 5], odd[16, unit] = np.nan, most
    odd[17] = 0.0
    odd[17, unit] = most
    got = run(odd)
    rest = [i for i in range(20) if i not in (3, 16, 17)]
    for k in got:
        assert np.array_equal(got[k][rest], clean[k][rest]), k
    assert np.isnan(got["logits"][3]).all() and np.isnan(got["value"][3])
    h = got["h_out"][[16, 17]].astype(np.float64)
    assert np.isfinite(h).all() and np.all(h[:, unit] == most)
    with np.errstate(all="raise"):
        logits = h @ w["pi_w"].astype(np.float64).T + w["pi_b"]
        value = h @ w["v_w"].astype(np.float64).ravel() + w["v_b"].ravel()
    # one term beyond all others: its product is rounded once and the others vanish behind it
    assert np.allclose(got["logits"][[16, 17]], logits, rtol=1e-6, atol=0)
    assert np.allclose(got["value"][[16, 17]], value, rtol=1e-6, atol=0)
    pol.close()


@pytest.mark.parametrize("kw,pipe", [(dict(heads=[63], rnn=64), "bf16x3"), (dict(heads=[64], rnn=64), "valu"),
                                     (dict(heads=[7], rnn=64, dtype="bf16"), "bf16"), (dict(heads=[7], rnn=48), "valu")])
def test_pipe_of_the_heads(torch_cuda, kw, pipe):
    """The arithmetic that the library reports for the heads' launch (the benchmark's peak follows it)."""
    net = dict(_BASE, fc=64, **kw)
    pol = binding.Policy(net, wl.weights(net), max_batch=3)
    assert pol.op_pipes()[-1] == pipe
    pol.close()
