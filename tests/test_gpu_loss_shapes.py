"""The loss kernels at the edges of their dispatch: one, two, four and eight trajectories per workgroup,
ragged last workgroups, partial sums added by the workgroups and by a second launch, 32 and 64 lanes per trajectory with partial chunks, 16-byte and element-wise
gradients, heads in every order of size, tiles too large for LDS with several trajectories or with one."""
import numpy as np
import pytest

from paper_2006_11751_amd import workloads as wl
from tests import parity
from tests.test_gpu_loss import RTOL, _ratios, _run

pytestmark = pytest.mark.gpu

FULL = (3, 3, 2, 2, 2, 8, 21)
CASES = [(FULL, 1, 1), (FULL, 32, 1023), (FULL, 32, 1024), (FULL, 31, 1027), (FULL, 33, 1026), (FULL, 65, 5),
         ((21, 1, 8), 7, 1025), ((4, 4), 5, 1030), ((2,) * 16, 40, 3), ((500,), 3, 1024), ((1000, 23), 2, 3),
         ((7,), 32, 1535), ((7,), 32, 1537), ((3, 3, 2, 2, 2, 11), 9, 1543), ((40, 9), 4, 1540), (FULL, 31, 639), (FULL, 31, 641),
         (FULL, 3, 256), (FULL, 3, 257), (FULL, 2, 512), (FULL, 2, 513), ((7,), 2, 4096), ((7,), 2, 4097),
         ((1,) * 16, 40, 1537), ((15,), 40, 511), ((15,), 40, 513), ((7,), 65, 1541), ((1200,), 3, 3)]


@pytest.mark.parametrize("heads,T,N", CASES, ids=["%s-%d-%d" % ("+".join(map(str, h)), t, n) for h, t, n in CASES])
def test_shapes(torch_cuda, ref, heads, T, N):
    hp = wl.loss_config(heads, T, N)
    tr = wl.trajectories(hp, 6100)
    g = _run(torch_cuda, hp, tr)
    o = ref.appo_loss(hp, **tr)
    for k in ("vs", "adv", "dvalues"):
        parity.assert_close(k, g[k], o[k], RTOL)
    scale = np.abs(o["loss"][:3]).max()
    assert np.all(np.abs(g["loss"] - o["loss"]) <= RTOL * (np.abs(o["loss"]) + scale)), (g["loss"], o["loss"])
    # (samples on a boundary of the clipping range may fall on either side in fp32)
    r, clip = _ratios(hp, tr), float(np.float32(hp["clip"]))
    sure = np.minimum(np.abs(r - clip), np.abs(r - 1.0 / clip)) > 1e-4
    parity.assert_close("dlogits", g["dlogits"][sure], o["dlogits"][sure], RTOL)
    again = _run(torch_cuda, hp, tr)
    for k in ("vs", "adv", "dvalues", "dlogits", "loss"):
        assert np.array_equal(g[k], again[k]), k


@pytest.mark.parametrize("heads,T", [((7,), 32), (FULL, 20), ((7,), 70), (FULL, 40), ((5,) * 15 + (3,), 40), ((150,), 40),
                                     ((200,), 32)], ids=lambda v: "+".join(map(str, v)) if isinstance(v, tuple) else None)
def test_trajectories_do_not_depend_on_their_number(torch_cuda, heads, T):
    """Targets and advantages of a trajectory are the same bits in every batch: with one, four or eight of
    them in a workgroup, and also where several do not fit LDS and one does (the kernel without LDS, with
    other exponentials, is for tiles that never fit)."""
    hp = wl.loss_config(heads, T, 1537)
    tr = wl.trajectories(hp, 6200)
    full = _run(torch_cuda, hp, tr)
    for n in (3, 511, 600, 1024):
        part = {k: np.ascontiguousarray(v[:, :n]) for k, v in tr.items()}
        g = _run(torch_cuda, dict(hp, N=n), part)
        for k in ("vs", "adv"):
            assert np.array_equal(g[k], full[k][:, :n]), (n, k)


@pytest.mark.parametrize("missing", ["vs", "adv", "loss", "workspace"])
def test_a_missing_buffer_is_refused_by_the_library(torch_cuda, missing):
    from paper_2006_11751_amd import binding
    hp = wl.loss_config((7,), 4, 3)
    tr = {k: torch_cuda.from_numpy(v).cuda() for k, v in wl.trajectories(hp).items()}
    out = dict(binding.appo_loss(hp, tr), **{missing: None})
    with pytest.raises(binding.SfError) as e:
        binding.appo_loss(hp, tr, out=out)
    assert e.value.code == binding.SF_ERR_ARG


@pytest.mark.parametrize("N", [1, 64, 300, 512])
def test_what_the_workspace_held_before_does_not_matter(torch_cuda, N):
    """The workgroups add their partial sums through the workspace without anything set there ahead: zeros,
    ones, random bits, and the entries of calls with other numbers of workgroups."""
    from paper_2006_11751_amd import binding
    t = torch_cuda
    hp = wl.loss_config(FULL, 4, N)
    tr = {k: t.from_numpy(v).cuda() for k, v in wl.trajectories(hp, 6300).items()}
    first = binding.appo_loss(hp, tr)
    want = first["loss"].cpu().numpy()
    assert np.all(np.isfinite(want))
    ws = first["workspace"]
    for fill in (0, 255, None, None):
        ws.copy_(t.randint(0, 256, ws.shape, device="cuda", dtype=t.uint8) if fill is None else t.full_like(ws, fill))
        for n in (N, max(1, N - 1), N):
            part = {k: v[:, :n].contiguous() for k, v in tr.items()}
            out = binding.appo_loss(dict(hp, N=n), part)
            out = dict(out, workspace=ws, loss=t.full((4,), float("nan"), device="cuda"))
            binding.appo_loss(dict(hp, N=n), part, out=out)
            got = out["loss"].cpu().numpy()
            assert np.array_equal(got, want) if n == N else np.all(np.isfinite(got)), (fill, n)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_losses_that_are_not_finite_are_written(torch_cuda, bad):
    hp = wl.loss_config((7,), 4, 9)
    tr = wl.trajectories(hp, 6400)
    tr["rewards"][2, 3] = bad
    g = _run(torch_cuda, hp, tr)
    again = _run(torch_cuda, hp, tr)
    assert not np.isfinite(g["loss"][1]) and np.isfinite(g["loss"][2])
    assert np.array_equal(g["loss"], again["loss"], equal_nan=True)
