"""The recurrent cell on bf16 features out of a ring in LDS (rnn_ring_kernel in k_rnn_bf16.hip): the bits of the
kernel that takes fp32 features (SF_FC_OUT_F32), for every tile, ragged rows, restarts, table rows that
are out of range, and K shorter and longer than the ring."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

SMALL = dict(obs=(3, 36, 64), dtype="bf16", p_done=0.2)
CASES = {  # network, rows of the handle, rows of the calls
    "gru-512": (2, dict(SMALL, fc=512, rnn=512), 2200, (1, 33, 65, 1024, 1025, 2048, 2049, 2200)),
    "lstm-512": (5, dict(SMALL, fc=128, rnn=512), 2200, (31, 1000, 1100, 2177)),
    "gru-64": (2, dict(SMALL, fc=64, rnn=64), 4200, (70, 4200)),
    "lstm-64": (5, dict(SMALL, fc=64, rnn=64), 4200, (63, 4129)),
}


@pytest.mark.parametrize("name", CASES)
def test_same_bits_as_on_fp32_features(torch_cuda, monkeypatch, name):
    torch = torch_cuda
    index, kw, rows, calls = CASES[name]
    net = wl.network(index, **dict(kw, name=name))
    w = wl.weights(net)
    g = torch.Generator(device="cuda").manual_seed(11)
    obs = torch.randint(0, 256, (rows,) + tuple(net["obs"]), generator=g, device="cuda", dtype=torch.uint8)
    table = 0.1 * torch.randn(2 * rows, wl.state_dim(net), generator=g, device="cuda")
    done = (torch.rand(rows, generator=g, device="cuda") < 0.2).byte()
    table[:rows][done != 0, 0] = float("nan")  # (a state that is not used)
    ids = torch.randperm(2 * rows, generator=g, device="cuda")[:rows].int()
    got = []
    for env in ({}, {"SF_FC_OUT_F32": "1"}):
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            pol = binding.Policy(net, w, max_batch=rows)
        out = []
        for B in calls:
            a = pol.step(obs[:B], table[:B], done[:B], 1, B)
            t = table.clone()
            i = ids[:B].clone()
            i[B // 2] = -1
            b = pol.step_indexed(obs[:B], t, i, done[:B], 1, B)
            torch.cuda.synchronize()
            out.append([a["h_out"].cpu().numpy(), a["logits"].cpu().numpy(), t.cpu().numpy(), b["logits"].cpu().numpy()])
        pol.close()
        got.append(out)
    for B, a, b in zip(calls, *got):
        for x, y in zip(a, b):
            assert np.array_equal(x, y, equal_nan=True), B
        assert np.isfinite(a[0]).all() and np.abs(a[0]).max() > 0.0
