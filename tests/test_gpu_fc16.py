"""The FC layer of 16-bit configurations on many rows (k_fc16.hip): the bits of the kernel that also takes
convolutions (SF_CONV_BF16_TC), for every tile of rows, ragged rows, and K shorter and longer than the ring of
chunks."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

PLAIN = dict(obs=(3, 36, 64), convs=[(16, 8, 4, 0), (32, 4, 2, 0)], fc=512, rnn=64, dtype="bf16", p_done=0.2)
LONG = dict(PLAIN, obs=(3, 72, 64))  # 21 chunks of 64
CASES = {  # network, rows of the handle (more than the kernel for few rows takes), rows of the calls
    "bf16-k576": (0, PLAIN, 2180, (1, 31, 33, 1024, 1025, 2047, 2049, 2180)),
    "bf16-k1344": (0, LONG, 2100, (5, 1500, 2100)),
    "fp16-k4608": (4, dict(fc=256), 4200, (3, 2049, 4200)),
}


@pytest.mark.parametrize("name", CASES)
def test_same_bits_as_the_convolution_kernel(torch_cuda, monkeypatch, name):
    torch = torch_cuda
    index, kw, rows, calls = CASES[name]
    net = wl.network(index, **dict(kw, name=name))
    w = wl.weights(net)
    g = torch.Generator(device="cuda").manual_seed(7)
    obs = torch.randint(0, 256, (rows,) + tuple(net["obs"]), generator=g, device="cuda", dtype=torch.uint8)
    h = 0.1 * torch.randn(rows, wl.state_dim(net), generator=g, device="cuda")
    done = (torch.rand(rows, generator=g, device="cuda") < 0.1).byte()
    got = []
    for env in ({}, {"SF_CONV_BF16_TC": "1"}):
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            pol = binding.Policy(net, w, max_batch=rows)
        out = []
        for B in calls:
            o = pol.step(obs[:B], h[:B], done[:B], 1, B)
            torch.cuda.synchronize()
            out.append({k: v.cpu().numpy().copy() for k, v in o.items()})
        pol.close()
        got.append(out)
    for B, a, b in zip(calls, *got):
        for k in a:
            assert np.array_equal(a[k], b[k]), (B, k)
        assert np.isfinite(a["logits"]).all() and np.abs(a["logits"]).max() > 0.0
