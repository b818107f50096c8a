"""Measurement layers (sf_meas.h, in the FC layer's launch or, hidden layers too large for that, their own): an infinite measurement, or an infinite hidden value, at every
place of a layer's inputs, against the oracle."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

N = 23  # four groups of threads take 5 or 6 of them each, eight loads at a time


def _net(hidden, dtype):
    return dict(name="meas", index=6, B=2 * N, obs=(3, 36, 64), encoder="conv", convs=[(16, 8, 4, 0), (32, 4, 2, 0)],
                fc=64, rnn=64, heads=[6], dtype=dtype, p_done=0.0, steps=1, obs_sub=0.0, obs_mul=wl.OBS_MUL,
                rnn_type="gru", meas_dim=N, meas_hidden=hidden)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("hidden", [[32], [64], [40, 32], [33, 64], [150, 64], [660, 32]])
def test_infinite_measurement(torch_cuda, ref, hidden, dtype, sign):
    """Rows 0 .. 22 hold an infinity at measurement 0 .. 22.  Each layer has one unit per input with a
    weight of the sign that makes it infinite; the others go to zero, so that one feature is infinite and the
    cell's gates are closed or open: the outputs are finite numbers."""
    torch = torch_cuda
    net = _net(hidden, dtype)
    w = wl.weights(net)
    for l, m in enumerate(w["meas_w"]):
        s = sign if l == 0 else 1
        m[:] = -s * np.abs(m)
        n = min(m.shape)
        m[np.arange(n), np.arange(n)] *= -1
    pol = binding.Policy(net, w)
    B, d = net["B"], pol.device
    obs, state, done, meas = wl.observations(net, 0), wl.initial_state(net), np.zeros(B, np.uint8), wl.measurements(net, 0)
    meas[np.arange(N), np.arange(N)] = sign * np.inf
    out = pol.step(*(torch.from_numpy(a).to(d) for a in (obs, state, done)), 7, 11, meas=torch.from_numpy(meas).to(d))
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        o = ref.policy_step(net, w, obs, state, done, 7, 11, meas=meas)
    assert np.isfinite(o["h_out"]).all()
    for k in ("h_out", "logits", "value"):
        parity.assert_close(k, out[k].cpu().numpy(), o[k], parity.RTOL[dtype])
    pol.close()
