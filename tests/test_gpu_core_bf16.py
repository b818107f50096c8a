"""The recurrent core of 16-bit configurations on either side of the rule that picks its kernel from
the handle's largest batch (k_dense_split.hip up to two rounds of its 32-row tile, k_rnn_bf16.hip
beyond): the features enter it as bf16 numbers on both; GRU and LSTM, with and without measurements,
beyond it."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

_SMALL = dict(obs=(3, 36, 64), dtype="bf16", fc=256, rnn=256)
# networks whose FC layer hands over fp32 numbers (256 units: the border is 1024 rows)
NETS = [wl.network(4, name="residual", **_SMALL),
        wl.network(6, name="measurements", meas_hidden=[40, 64], **_SMALL),
        wl.network(5, name="lstm_measurements", meas_dim=9, meas_hidden=[128], **_SMALL)]


def _run(torch, pol, net, B):
    d = pol.device
    t = lambda a: None if a is None else torch.from_numpy(a).to(d)
    out = pol.step(t(wl.observations(net, 0, B)), t(wl.initial_state(net, B)), t(wl.done_mask(net, 0, B)), 7, 11,
                   meas=t(wl.measurements(net, 0, B)))
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("net", NETS, ids=lambda n: n["name"])
def test_both_kernels_round_the_features(torch_cuda, net):
    """The same row from a small handle and from a large one.  What may differ: the order of the
    sums, one rounding of the state (2^-17 of it), and, where another order of the FC layer's sum
    moves a feature over a rounding border (a few in 10^4 features), 2^-8 of that feature.  Features
    with all their bits on one side would differ by 2^-10 of every feature: about 2e-3 of the result."""
    w = wl.weights(net)
    got = []
    for max_batch in (100, 1100):
        pol = binding.Policy(net, w, max_batch=max_batch)
        got.append(_run(torch_cuda, pol, net, 100))
        pol.close()
    for k in ("h_out", "logits", "value"):
        a, b = (g[k].astype(np.float64) for g in got)
        assert np.linalg.norm(a - b) <= 3e-4 * np.linalg.norm(b), k


@pytest.mark.parametrize("rnn_type", ["gru", "lstm"])
def test_rounding_before_or_inside_the_core(torch_cuda, monkeypatch, rnn_type):
    """The FC layer hands over bf16 numbers, or (by the switch) fp32 ones that the core rounds: the
    same bits, in each of its tiles (16 x 8, 32 x 8, 32 x 16)."""
    net = wl.network(2, name="features", obs=(3, 36, 64), fc=128, rnn=128, rnn_type=rnn_type)
    w = wl.weights(net)
    for B in (1, 40, 300, 600):
        pol = binding.Policy(net, w, max_batch=B)
        a = _run(torch_cuda, pol, net, B)
        pol.close()
        with monkeypatch.context() as m:
            m.setenv("SF_FC_OUT_F32", "1")
            pol = binding.Policy(net, w, max_batch=B)
        b = _run(torch_cuda, pol, net, B)
        pol.close()
        for k in a:
            assert np.array_equal(a[k], b[k]), (B, k)


# 512 hidden units: up to 512 rows k_dense_split.hip, from 513 on k_rnn_bf16.hip
LARGE = [wl.network(2, name="gru", obs=(3, 36, 64), fc=64, rnn=512),
         wl.network(5, name="lstm", obs=(3, 36, 64), dtype="bf16", fc=128, rnn=512),
         wl.network(6, name="gru_measurements", obs=(3, 36, 64), dtype="bf16", fc=64, rnn=512, meas_hidden=[40, 64]),
         wl.network(5, name="lstm_measurements", obs=(3, 36, 64), dtype="bf16", fc=64, rnn=512, meas_dim=9, meas_hidden=[128])]


@pytest.mark.parametrize("net", LARGE, ids=lambda n: n["name"])
def test_many_rows(torch_cuda, ref, net):
    """Handles beyond the rule, on ragged batches: the oracle's result, for the plain and the indexed
    step, and not the bits of the other kernel (which would mean that this one was not run)."""
    torch = torch_cuda
    w = wl.weights(net)
    B, n_env = 137, 300
    small = binding.Policy(net, w, max_batch=512)
    other = _run(torch, small, net, B)
    small.close()
    pol = binding.Policy(net, w, max_batch=513)
    g = _run(torch, pol, net, B)
    assert not np.array_equal(g["h_out"], other["h_out"])
    obs, state, done, meas = wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B), wl.measurements(net, 0, B)
    parity.check_against_oracle(net, g, ref.policy_step(net, w, obs, state, done, 7, 11, meas=meas), ref, 7, 11)
    table = wl.initial_state(net, n_env)
    ids = np.random.default_rng(5).permutation(n_env)[:B].astype(np.int32)
    t = lambda a: None if a is None else torch.from_numpy(a).to(pol.device)
    plain = pol.step(t(obs), t(table[ids]), t(done), 7, 11, meas=t(meas))
    t_gpu = t(table)
    pol.step_indexed(t(obs), t_gpu, t(ids), t(done), 7, 11, meas=t(meas))
    torch.cuda.synchronize()
    table[ids] = plain["h_out"].cpu().numpy()
    assert np.array_equal(t_gpu.cpu().numpy(), table)
    full = _run(torch, pol, net, 513)
    for k in g:
        assert np.array_equal(full[k][:B], g[k]), k
    pol.close()
