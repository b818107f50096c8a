"""The first two convolutions of an fp32 network in one launch (k_conv12_split.hip) against the two separate
launches and the oracle: one and several frames per workgroup, a frame height that leaves rows over, frames
at an address that is a multiple of four bytes only, a graph recorded before an update that the second layer's
split does not take."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("height", [72, 75])
def test_one_launch_and_two(torch_cuda, ref, monkeypatch, height):
    torch = torch_cuda
    net = wl.network(1, fc=64, rnn=64, name="conv12_split", obs=(3, height, 128))
    w = wl.weights(net)
    B = 2060  # eight and nine frames per workgroup; enough for the frame-resident kernel of the first layer alone
    one = binding.Policy(net, w, max_batch=B)
    with monkeypatch.context() as m:
        m.setenv("SF_NO_CONV12_FUSE", "1")
        two = binding.Policy(net, w, max_batch=B)
    assert one.op_kernels()[:2] == ["conv12_split"] * 2 and two.op_kernels()[:2] == ["conv1_i8", "conv_image_split"]
    o_, s_, d_ = wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B)
    raw = torch.empty(o_.size + 4, dtype=torch.uint8, device="cuda")
    shifted = raw[4:].view(o_.shape).copy_(torch.from_numpy(o_))
    obs, st, dn = (torch.from_numpy(a).cuda() for a in (o_, s_, d_))
    step = lambda pol, n, x: {k: v.cpu().numpy() for k, v in pol.step(x[:n], st[:n], dn[:n], 7, 11).items()}
    full, apart, moved = step(one, B, obs), step(two, B, obs), step(one, B, shifted)
    rows = np.array([0, 1, 255, 256, 257, 511, 512, 599, 2047, 2059])
    want = ref.policy_step(net, w, o_[rows], s_[rows], d_[rows], 7, 11)
    for k in ("logits", "value", "h_out"):
        parity.assert_close(k, full[k][rows], want[k], 1e-4)
        # the same products in another order: a few roundings of an fp32 sum of 512 terms, then of the rest
        assert np.abs(full[k] - apart[k]).max() <= 2e-5 * np.abs(apart[k]).max(), k
        assert np.array_equal(moved[k], full[k]), k  # (a frame's bits do not depend on its address)
    # a frame's bits depend neither on the batch nor on whether one, two or four workgroups share it
    for n in (600, 385, 384, 257, 256, 129, 128, 65, 64, 1):
        for x in (obs, shifted):
            part = step(one, n, x)
            for k in full:
                assert np.array_equal(part[k], full[k][:n]), (n, k)
    # the second layer is in the first one's launch
    for pol in (one, two):
        pol.set_op_timing(True)
        step(pol, 300, obs)
        ms = pol.last_op_times_ms()
        assert (ms[1] == 0.0) == (pol is one) and min(ms[:1] + ms[2:]) > 0.0, ms
        pol.set_op_timing(False)
    one.close()
    two.close()


@pytest.mark.parametrize("B", [37, 300, 600])
def test_recorded_step_whose_second_layer_is_refused(torch_cuda, ref, B):
    """A graph keeps the one launch; with parameters that the second layer's split does not take, it computes
    that layer in fp32: frames shared by four and by two workgroups, and several whole frames per workgroup."""
    torch = torch_cuda
    net = wl.network(1, fc=64, rnn=64, name="conv12_recorded")
    w = wl.weights(net)
    huge = {k: [a.copy() for a in v] if isinstance(v, list) else v.copy() for k, v in w.items()}
    huge["conv_w"][0] *= np.float32(2.0 ** 110)
    huge["conv_b"][0] *= np.float32(2.0 ** 110)
    huge["conv_w"][1] *= np.float32(2.0 ** -110)
    pol = binding.Policy(net, w, max_batch=B)
    assert pol.op_kernels()[0] == "conv12_split"
    o_, s_, d_ = wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B)
    obs, st, dn = (torch.from_numpy(a).cuda() for a in (o_, s_, d_))
    out = pol.step(obs, st, dn, 7, 11)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pol.step(obs, st, dn, 7, 11, out=out, stream=torch.cuda.current_stream())
    pol.update_weights(huge)
    assert pol.op_kernels()[:2] == ["conv1_i8", "gemm_mfma"]
    rows = np.unique(np.array([0, 1, B // 3, B // 2, B - 2, B - 1]))
    want = ref.policy_step(net, huge, o_[rows], s_[rows], d_[rows], 7, 11)
    for _ in range(2):
        for v in out.values():
            v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        recorded = {k: v.cpu().numpy() for k, v in out.items()}
        for k in ("logits", "value", "h_out"):
            parity.assert_close(k, recorded[k][rows], want[k], 1e-4)
        eager = {k: v.cpu().numpy() for k, v in pol.step(obs, st, dn, 7, 11).items()}  # (the fp32 kernel)
        for k in ("logits", "value", "h_out"):
            parity.assert_close(k, recorded[k], eager[k], 1e-4)
    pol.close()


@pytest.mark.parametrize("height", [72, 74])
def test_bf16_frames_shared_by_workgroups(torch_cuda, height):
    """The same of the bf16 network, whose one launch gives the bits of the two separate kernels
    (test_gpu_parity.py)."""
    torch = torch_cuda
    net = wl.network(2, fc=64, rnn=64, name="conv12_bf16", obs=(3, height, 128))
    B = 300
    pol = binding.Policy(net, wl.weights(net), max_batch=B)
    assert pol.op_kernels()[0] == "conv12_fused"
    obs, st, dn = (torch.from_numpy(a).cuda() for a in (wl.observations(net, 0, B), wl.initial_state(net, B),
                                                       wl.done_mask(net, 0, B)))
    step = lambda n: {k: v.cpu().numpy() for k, v in pol.step(obs[:n], st[:n], dn[:n], 7, 11).items()}
    full = step(B)
    for n in (257, 256, 129, 128, 65, 64, 1):
        part = step(n)
        for k in full:
            assert np.array_equal(part[k], full[k][:n]), (n, k)
    pol.close()
