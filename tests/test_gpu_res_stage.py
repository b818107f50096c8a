"""32-channel stages of the residual encoder in one launch: one to three tiles per wave with the filter
banks in LDS, and the stages whose banks do not fit there (three blocks, wide frames)."""
import numpy as np
import pytest

from paper_2006_11751_amd import binding, workloads as wl
from tests import parity
from tests.test_gpu_parity import RESNET_BF16_SMALL, _gpu_step

pytestmark = pytest.mark.gpu

# second stage frames (32 channels): 8 x 32 (one tile per wave), 12 x 32 with a ragged wave, 18 x 32 (three),
# 11 x 16; 600 frames: several per workgroup; 131 frames of 13 x 16, stacked by two; up to 128 and 64 frames:
# two and four strips per frame; three blocks: the kernel that streams its banks
CASES = [((3, 32, 128), 2, 5), ((3, 45, 128), 2, 600), ((3, 72, 128), 1, 259), ((3, 44, 64), 2, 13),
         ((3, 72, 128), 3, 3), ((3, 24, 256), 2, 4),
         ((3, 100, 128), 2, 131), ((3, 72, 128), 2, 128), ((3, 72, 128), 2, 64), ((3, 71, 64), 1, 70), ((3, 41, 128), 2, 1)]


@pytest.mark.parametrize("obs,blocks,B", CASES, ids=["%dx%d-%d-%d" % (o[1], o[2], n, b) for o, n, b in CASES])
def test_stage_with_its_banks_in_lds(torch_cuda, ref, monkeypatch, obs, blocks, B):
    torch = torch_cuda
    net = dict(RESNET_BF16_SMALL, name="res_stage_%dx%d" % obs[1:], B=B, obs=obs, blocks_per_stage=blocks)
    if blocks == 3:  # (at most 20 convolutions)
        net["stages"] = [16, 32]
    w = wl.weights(net)
    o_, h_, d_ = wl.observations(net, 0, B), wl.initial_state(net, B), wl.done_mask(net, 0, B)
    pol = binding.Policy(net, w)
    assert "res_stage" in pol.op_kernels(), pol.op_kernels()
    g = _gpu_step(torch, pol, o_, h_, d_, 7, 11)
    pol.close()
    rows = np.unique(np.array([0, B // 2, B - 1]))
    o = ref.policy_step(net, w, o_[rows], h_[rows], d_[rows], 7, 11)
    monkeypatch.setenv("SF_NO_RES_STAGE", "1")
    old = binding.Policy(net, w)
    monkeypatch.delenv("SF_NO_RES_STAGE")
    g2 = _gpu_step(torch, old, o_, h_, d_, 7, 11)
    old.close()
    if B > 64:  # (shared among workgroups or not, a frame has the same bits)
        pol = binding.Policy(net, w)
        for n in (min(128, B - 1), 64, 3):
            part = _gpu_step(torch, pol, o_[:n], h_[:n], d_[:n], 7, 11)
            for k in ("h_out", "value", "logits"):
                assert np.array_equal(part[k], g[k][:n]), (n, k)
        pol.close()
    for k in ("h_out", "value"):
        parity.assert_close(k, g[k][rows], o[k], 1e-2)
        # (fp16 streams rounded at different points, each about 1e-3 from the oracle)
        parity.assert_close(k + " vs per-block kernels", g[k], g2[k], 1e-2)


# first stage frames (16 channels): rows that the waves share unevenly in four, two and one column groups; the fewest
# that are taken (one row per wave at 16 columns: strips leave waves without any); three blocks, and several frames
# per workgroup
CASES16 = [((3, 34, 128), 2, 5), ((3, 10, 128), 1, 4), ((3, 71, 128), 2, 300), ((3, 45, 64), 2, 261), ((3, 37, 32), 2, 3),
           ((3, 32, 32), 2, 270), ((3, 33, 32), 1, 64), ((3, 45, 64), 3, 260), ((3, 71, 128), 3, 2)]


@pytest.mark.parametrize("obs,blocks,B", CASES16, ids=["%dx%d-%d-%d" % (o[1], o[2], n, b) for o, n, b in CASES16])
def test_rows_of_a_column_group(torch_cuda, ref, monkeypatch, obs, blocks, B):
    test_stage_with_its_banks_in_lds(torch_cuda, ref, monkeypatch, obs, blocks, B)


@pytest.mark.parametrize("obs,blocks", [((3, 32, 32), 1), ((3, 40, 64), 2), ((3, 72, 128), 2), ((3, 32, 64), 3)])
def test_order_of_the_taps(torch_cuda, ref, obs, blocks):
    """The products of a 16-channel convolution are added in the order (0, 1), (3, 4), (6, 7), (2, 5), (8): a small
    one of tap 5 is kept if the large ones of taps 4 and 7, which cancel, are both there before it."""
    net = dict(RESNET_BF16_SMALL, name="taps_%dx%d" % obs[1:], B=3, obs=obs, stages=[16], blocks_per_stage=blocks)
    w = wl.weights(net)
    w["conv_w"] = [np.zeros_like(a) for a in w["conv_w"]]
    w["conv_b"] = [np.zeros_like(b) for b in w["conv_b"]]
    w["conv_b"][0][:] = 1.0  # every pixel is 1, and a multiple of 2^-9 below 2 behind each block
    for k in range(blocks):
        a, b = w["conv_w"][1 + 2 * k], w["conv_w"][2 + 2 * k]
        a[0, 0, 1, 1], a[0, 0, 2, 1], a[0, 0, 1, 2] = -2.0 ** 14, 2.0 ** 14, 2.0 ** -13
        b[:, 0, 1, 1] = 2.0 ** 10
    o_, h_, d_ = wl.observations(net, 0, 3), wl.initial_state(net, 3), wl.done_mask(net, 0, 3)
    pol = binding.Policy(net, w)
    assert "res_stage" in pol.op_kernels(), pol.op_kernels()
    g = _gpu_step(torch_cuda, pol, o_, h_, d_, 7, 11)
    pol.close()
    o = ref.policy_step(net, w, o_, h_, d_, 7, 11)
    for k in ("h_out", "value"):
        parity.assert_close(k, g[k], o[k], 1e-2)
