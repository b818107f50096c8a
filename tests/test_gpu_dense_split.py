"""FC layer and recurrent cell on operands split into bf16 terms (k_dense_split.hip): the tiles'
edges, waves without a K step, a measurement piece in the middle of K, the kernel for many rows,
gathered states, and states that hold an infinity or a NaN.  Against the oracle where a sum is
computed, bit for bit where only the place of a row differs (its sums run in an order that K alone
decides)."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

_BASE = dict(obs=(3, 36, 64), encoder="conv", convs=[(16, 8, 4, 0), (32, 4, 2, 0)], dtype="fp32", p_done=0.3, steps=1,
             obs_sub=0.0, obs_mul=wl.OBS_MUL, meas_dim=0, meas_hidden=[], rnn_type="gru", heads=[6], index=5)


def _net(**kw):
    n = dict(_BASE, **kw)
    n["name"] = "dense"
    return n


# (network, max_batch, batch sizes).  512 hidden units: one round of 16 x 8, 32 x 8, 32 x 16, 32 x 32 tiles up
# to 64, 128, 256, 512 rows; the kernel for many rows from max_batch 513 on (64 rows x 32 units).
CASES = [
    (_net(fc=512, rnn=512), 512, [1, 16, 17, 64, 65, 128, 129, 257, 512]),
    (_net(fc=512, rnn=512), 513, [1, 64, 65, 513]),
    (_net(fc=128, rnn=512, rnn_type="lstm"), 300, [15, 100, 300]),
    (_net(fc=256, rnn=512, rnn_type="lstm"), 600, [600]),
    (_net(fc=128, rnn=512, meas_dim=5, meas_hidden=[128]), 520, [520]),      # many rows, three pieces of K
    (_net(fc=96, rnn=512, meas_dim=5, meas_hidden=[32]), 520, [70, 520]),    # pieces that are no chunk of four K steps
    (_net(fc=32, rnn=32), 40, [40]),                                         # two K steps for eight waves
    (_net(fc=32, rnn=32, rnn_type="lstm"), 3, [3]),
    (_net(fc=128, rnn=128, dtype="bf16"), 70, [1, 70]),
    (_net(fc=128, rnn=128, rnn_type="lstm", dtype="bf16", meas_dim=5, meas_hidden=[64]), 33, [33]),
    (_net(fc=64, rnn=96, dtype="bf16"), 50, [50]),
    # the FC layer's tiles: 512 outputs, one round of 32 x 32, 32 x 64, 64 x 64 up to 512, 1024, 2048 rows;
    # outputs that are no multiple of 64
    (_net(fc=512, rnn=32), 2600, [512, 513, 1024, 1025, 2048, 2049, 2600]),
    (_net(fc=512, rnn=32, dtype="bf16"), 2048, [128, 129, 512, 513, 1024, 1025, 2048]),
    (_net(fc=544, rnn=32), 500, [480, 481, 500]),
    (_net(fc=544, rnn=32, dtype="bf16"), 500, [480, 481, 500]),
]


def _run(torch, pol, net, obs, state, done, meas):
    d = pol.device
    t = lambda a: None if a is None else torch.from_numpy(a).to(d)
    out = pol.step(t(obs), t(state), t(done), 7, 11, meas=t(meas))
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("net,max_batch,sizes", CASES,
                         ids=lambda v: "%s%d+%d-%d-%s" % (v["rnn_type"], v["fc"], sum(v["meas_hidden"]), v["rnn"], v["dtype"])
                         if isinstance(v, dict) else None)
def test_tiles(torch_cuda, ref, net, max_batch, sizes):
    torch = torch_cuda
    w = wl.weights(net)
    pol = binding.Policy(net, w, max_batch=max_batch)
    B = max(sizes)
    obs, state, done, meas = (wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B),
                              wl.measurements(net, 0, B))
    o = ref.policy_step(net, w, obs, state, done, 7, 11, meas=meas)
    full = None
    for n in sorted(sizes, reverse=True):
        g = _run(torch, pol, net, obs[:n], state[:n], done[:n], None if meas is None else meas[:n])
        if full is None:
            full = g
            parity.check_against_oracle(net, g, o, ref, 7, 11)
        for k in g:  # another tile, the same bits
            assert np.array_equal(g[k], full[k][:n]), (n, k)
    pol.close()


@pytest.mark.parametrize("max_batch,B", [(64, 64), (256, 200), (300, 300), (600, 600)])
@pytest.mark.parametrize("rnn_type", ["gru", "lstm"])
def test_gathered_states(torch_cuda, max_batch, B, rnn_type):
    """Rows that index a state table give the bits of the plain step; an id outside the table
    that of a reset row."""
    torch = torch_cuda
    net = _net(fc=128, rnn=512, rnn_type=rnn_type)
    pol = binding.Policy(net, wl.weights(net), max_batch=max_batch)
    d, n_env = pol.device, 2 * B
    obs, done = wl.observations(net, 0, B), wl.done_mask(net, 0, B)
    table = wl.initial_state(net, n_env)
    ids = np.random.default_rng(5).permutation(n_env)[:B].astype(np.int32)
    ids[3], ids[B - 1] = n_env, -1
    ok = (ids >= 0) & (ids < n_env)
    state = np.where(ok[:, None], table[np.where(ok, ids, 0)], 0).astype(np.float32)
    plain = _run(torch, pol, net, obs, state, done, None)
    t_gpu = torch.from_numpy(table).to(d)
    pol.step_indexed(torch.from_numpy(obs).to(d), t_gpu, torch.from_numpy(ids).to(d), torch.from_numpy(done).to(d), 7, 11)
    torch.cuda.synchronize()
    assert np.array_equal(t_gpu.cpu().numpy()[ids[ok]], plain["h_out"][ok])
    pol.close()


@pytest.mark.parametrize("max_batch,B", [(40, 40), (200, 200), (300, 300), (600, 600)])
@pytest.mark.parametrize("rnn_type", ["gru", "lstm"])
def test_states_without_terms(torch_cuda, ref, max_batch, B, rnn_type):
    """An infinity, a NaN and a number that would round up to an infinity in bf16: their rows
    follow the definition, the others keep their bits."""
    torch = torch_cuda
    net = _net(fc=128, rnn=512, rnn_type=rnn_type)
    w = wl.weights(net)
    pol = binding.Policy(net, w, max_batch=max_batch)
    obs, state = wl.observations(net, 0, B), wl.initial_state(net, B)
    done = np.zeros(B, np.uint8)
    done[5] = 1
    clean = _run(torch, pol, net, obs, state, done, None)
    odd = {1: np.inf, 5: np.nan, 17: -np.inf, B - 1: np.finfo(np.float32).max, 33: np.nan}
    for row, v in odd.items():
        state[row, 3 * row % 512] = v
    got = _run(torch, pol, net, obs, state, done, None)
    rest = [i for i in range(B) if i not in odd or i == 5]  # (row 5 is reset: its state is not read)
    assert np.array_equal(got["h_out"][rest], clean["h_out"][rest])
    with np.errstate(all="ignore"):
        o = ref.policy_step(net, w, obs, state, done, 7, 11)
    for row in (1, 17, B - 1):
        a, b = got["h_out"][row].astype(np.float64), o["h_out"][row].astype(np.float64)
        assert np.array_equal(np.isfinite(a), np.isfinite(b)), row
        # (GRU, infinity: a closed r gate times an infinite sum is a NaN, in about half of the units)
        m = np.isfinite(b) & (np.abs(b) < 1e30)
        assert m.sum() >= 200 and np.max(np.abs(a[m] - b[m])) < 1e-4, row
    assert np.isnan(got["h_out"][33]).all()
    pol.close()


@pytest.mark.parametrize("max_batch", [40, 200, 600])
@pytest.mark.parametrize("rnn_type", ["gru", "lstm"])
def test_sums_that_overflow(torch_cuda, ref, max_batch, rnn_type):
    """Finite operands whose products overflow: the infinity of the definition, in the FC layer, in a cell
    and in the heads, and not the NaN that terms of both signs would add up to."""
    torch = torch_cuda
    B = max_batch
    net = _net(fc=128, rnn=512, rnn_type=rnn_type)
    w = wl.weights(net)
    obs, state, done = wl.observations(net, 0, B), wl.initial_state(net, B), np.zeros(B, np.uint8)
    # FC: activations of 2^118, one unit with positive weights only, the others go to zero
    v = {k: [a.copy() for a in x] if isinstance(x, list) else x.copy() for k, x in w.items()}
    v["conv_w"][1] *= np.float32(2.0 ** 118)
    v["conv_b"][1] *= np.float32(2.0 ** 118)
    v["fc_w"] = -np.abs(v["fc_w"]) * np.float32(2.0 ** 24)
    v["fc_w"][17] *= -1
    # cell: a state of 2^127 in one place (with an open r gate everywhere, so that no unit is 0 * infinity,
    # and at that unit an open z gate), and zero there in the other rows
    u = {k: [a.copy() for a in x] if isinstance(x, list) else x.copy() for k, x in w.items()}
    c, H, rows = 77, 512, np.array([0, 15, 16, B - 1])
    u["rnn_w_hh"][:, c] *= np.float32(2.0 ** 16)
    if rnn_type == "gru":
        u["rnn_w_hh"][:H, c] = np.abs(u["rnn_w_hh"][:H, c])
        u["rnn_w_hh"][H + c, c] = np.abs(u["rnn_w_hh"][H + c, c])
        u["pi_w"][:, c] *= np.float32(2.0 ** 16)
        u["v_w"][c] = 2.0 ** 16
    big = state.copy()
    big[:, c] = 0
    big[rows, c] = 1.703 * 2.0 ** 127
    for weights, st in ((v, state), (u, big)):
        pol = binding.Policy(net, weights, max_batch=max_batch)
        g = _run(torch, pol, net, obs, st, done, None)
        pol.close()
        with np.errstate(all="ignore"):
            o = ref.policy_step(net, weights, obs, st, done, 7, 11)
        for k in ("h_out", "logits", "value"):
            a, b = g[k].astype(np.float64), o[k].astype(np.float64)
            m = np.isfinite(b) & (np.abs(b) < 1e30)
            assert np.array_equal(a[~m], b[~m]), k
            # (heads with weights of 2^16: what they make of a state's last bits is not looked at)
            assert (weights is u and k != "h_out") or np.max(np.abs(a[m] - b[m])) < 1e-4, k
    if rnn_type == "gru":
        assert np.isinf(o["logits"][rows]).all() and np.isfinite(o["logits"]).sum() == (B - 4) * 6


@pytest.mark.parametrize("rnn_type", ["gru", "lstm"])
def test_few_rows_of_a_handle_for_many(torch_cuda, ref, rnn_type):
    """The kernel for many rows on 16, 32 and 64 rows per workgroup: one round of them up to 256 and 512 rows of 512
    hidden units; gathered states, and rows whose sums are computed by the definition."""
    test_tiles(torch_cuda, ref, _net(fc=128, rnn=512, rnn_type=rnn_type), 600, [1, 16, 17, 255, 256, 257, 511, 512, 513, 600])
    for B in (200, 400):
        test_gathered_states(torch_cuda, 600, B, rnn_type)
        test_states_without_terms(torch_cuda, ref, 600, B, rnn_type)
