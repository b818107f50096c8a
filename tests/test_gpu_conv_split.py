"""fp32 convolutions on operands split into two fp16 terms (k_conv_image_split.hip): rounds of one
and two frames with a ragged last one, several rounds per workgroup, another frame size, channels of
very different size, and the admission test that sends a layer back to the fp32 kernel."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def _run(torch, pol, net, B, w_obs=0):
    d = pol.device
    obs, state, done = wl.observations(net, w_obs, B), wl.initial_state(net, B), wl.done_mask(net, w_obs, B)
    out = pol.step(torch.from_numpy(obs).to(d), torch.from_numpy(state).to(d), torch.from_numpy(done).to(d), 7, 11)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}, (obs, state, done)


def _net(**kw):
    return wl.network(1, fc=64, rnn=64, name="conv_split", **kw)


@pytest.mark.parametrize("obs,kernels", [((3, 72, 128), ["conv_image_split", "conv_image_split"]),
                                         ((3, 68, 132), ["conv_image_split", "gemm_mfma"])])
def test_rounds_and_frame_sizes(torch_cuda, ref, obs, kernels):
    torch = torch_cuda
    net = _net(obs=obs)
    w = wl.weights(net)
    pol = binding.Policy(net, w, max_batch=1100)
    assert pol.op_kernels()[1:3] == kernels
    full = None
    for B in (1100, 515, 3, 2, 1):  # 1100 frames: three and two rounds per workgroup
        g, (o_, s_, d_) = _run(torch, pol, net, B)
        if full is None:
            full = g
            rows = np.array([0, 1, 2, 511, 512, 513, 1023, 1024, 1097, 1098, 1099])
            o = ref.policy_step(net, w, o_[rows], s_[rows], d_[rows], 7, 11)
            for k in ("logits", "value", "h_out"):
                parity.assert_close(k, g[k][rows], o[k], 1e-4)
        for k in g:
            assert np.array_equal(g[k], full[k][:B]), (B, k)
    pol.close()


@pytest.mark.parametrize("spread", [0, 12, 40])
def test_channels_of_different_size(torch_cuda, ref, spread):
    """Channel c of a layer 2^s larger and the next layer's weights on it 2^s smaller: the network
    is the same, and the split's errors follow each channel's own size."""
    torch = torch_cuda
    net = _net()
    w = wl.weights(net)
    rng = np.random.default_rng(3)
    for l in (0, 1):
        s = np.exp2(rng.integers(-spread, spread + 1, w["conv_w"][l].shape[0])).astype(np.float32)
        w["conv_w"][l] = w["conv_w"][l] * s[:, None, None, None]
        w["conv_b"][l] = w["conv_b"][l] * s
        w["conv_w"][l + 1] = w["conv_w"][l + 1] / s[None, :, None, None]
    pol = binding.Policy(net, w, max_batch=33)
    assert pol.op_kernels()[1:3] == ["conv_image_split"] * 2
    g, (o_, s_, d_) = _run(torch, pol, net, 33)
    parity.check_against_oracle(net, g, ref.policy_step(net, w, o_, s_, d_, 7, 11), ref, 7, 11)
    pol.close()


def test_admission_follows_the_parameters(torch_cuda, ref):
    """Activations near the end of fp32's range go to the fp32 kernel; a weight update moves the
    layer there and back, each state with the bits of a fresh policy."""
    torch = torch_cuda
    net = _net()
    w = wl.weights(net)
    huge = {k: [a.copy() for a in v] if isinstance(v, list) else v.copy() for k, v in w.items()}
    huge["conv_w"][0] *= np.float32(2.0 ** 110)
    huge["conv_b"][0] *= np.float32(2.0 ** 110)
    huge["conv_w"][1] *= np.float32(2.0 ** -110)
    pol = binding.Policy(net, w, max_batch=5)
    first, _ = _run(torch, pol, net, 5)
    pol.update_weights(huge)
    assert pol.op_kernels()[1:3] == ["gemm_mfma", "conv_image_split"]
    g, (o_, s_, d_) = _run(torch, pol, net, 5)
    parity.check_against_oracle(net, g, ref.policy_step(net, huge, o_, s_, d_, 7, 11), ref, 7, 11)
    pol.update_weights(w)
    assert pol.op_kernels()[1:3] == ["conv_image_split"] * 2
    again, _ = _run(torch, pol, net, 5)
    for k in first:
        assert np.array_equal(first[k], again[k]), k
    pol.close()


@pytest.mark.parametrize("factor", [-110, 110])
def test_recorded_step_after_an_update(torch_cuda, ref, factor):
    """A graph keeps its kernels: recorded with the split admitted and replayed with parameters for
    which it is not (factor < 0: the other way round), it computes the new parameters' network."""
    torch = torch_cuda
    net = _net()
    w = wl.weights(net)
    huge = {k: [a.copy() for a in v] if isinstance(v, list) else v.copy() for k, v in w.items()}
    huge["conv_w"][0] *= np.float32(2.0 ** 110)
    huge["conv_b"][0] *= np.float32(2.0 ** 110)
    huge["conv_w"][1] *= np.float32(2.0 ** -110)
    before, after = (w, huge) if factor > 0 else (huge, w)
    B = 37
    pol = binding.Policy(net, before, max_batch=B)
    o_, s_, d_ = wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B)
    obs, st, dn = (torch.from_numpy(a).cuda() for a in (o_, s_, d_))
    out = pol.step(obs, st, dn, 7, 11)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pol.step(obs, st, dn, 7, 11, out=out, stream=torch.cuda.current_stream())
    pol.update_weights(after)
    torch.cuda.synchronize()
    want = ref.policy_step(net, after, o_, s_, d_, 7, 11)
    for _ in range(3):
        for v in out.values():
            v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for k in ("logits", "value", "h_out"):
            parity.assert_close(k, out[k].cpu().numpy(), want[k], 1e-4)
    pol.close()
