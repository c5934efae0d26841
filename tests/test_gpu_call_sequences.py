"""Calls that follow one another on the same workspace or change the
process-wide setting: each gives what it would give alone."""
import json

import numpy as np
import pytest
import torch

from parity_util import device_inputs, workspace_for
from test_gpu_parity import small_workload

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2501_04782_amd import raster


def same_gradients(a, b):
    return [k for k, g in a.items() if g is not None and not torch.equal(g, b[k])]


@pytest.mark.parametrize("n", [3000, 40000])
def test_inspection_between_forward_and_backward(n):
    """gv_project_fwd with the same frame on the workspace of a forward leaves
    what the backward needs: the same gradients bit for bit."""
    w = small_workload(11, 640, 400, n, 1, trajectory=True, z=(2.0, 6.0), ls=(-4.0, 0.4))
    scene, cam, poses, times = device_inputs(w)
    ws = workspace_for(scene, cam, poses, times, margin=3.0)
    pose = poses[0].contiguous()
    dl = torch.from_numpy(np.random.default_rng(1).normal(0, 1, (3, 400, 640)).astype(np.float32)).cuda()
    img = raster.render_fwd(scene, cam, pose, 0.0, ws)
    want, dpose = raster.render_bwd(scene, cam, pose, 0.0, ws, img, dL_dimage=dl)
    for _ in range(3):
        img = raster.render_fwd(scene, cam, pose, 0.0, ws)
        raster.project_fwd(scene, cam, pose, 0.0, ws)
        got, dp = raster.render_bwd(scene, cam, pose, 0.0, ws, img, dL_dimage=dl)
        torch.cuda.synchronize()
        assert same_gradients(want, got) == [] and torch.equal(dpose, dp)


def test_autotuned_choice_runs_as_measured(tmp_path):
    """A setting that gv_autotune finds (here in its cache, so that it is known)
    runs as it was measured on launches of the size it was tuned on, also where
    the defaults would take the quadrant kernels; saving it with get_tuning and
    setting it again after another restores it, on smaller launches too.
    Gradient bits tell the kernels apart (order of sums)."""
    w = small_workload(13, 96, 64, 1500, 4, trajectory=True)
    scene, cam, poses, times = device_inputs(w)
    ws = workspace_for(scene, cam, poses, times)
    dl = torch.from_numpy(np.random.default_rng(2).normal(0, 1, (4, 3, 64, 96)).astype(np.float32)).cuda()

    def bits(frames=4):
        return raster.render_batch(scene, cam, poses[:frames], times[:frames], ws, dL_dimages=dl[:frames])["grads"]

    cache = tmp_path / "tune.jsonl"
    old = raster.get_tuning()
    try:
        quadrant = bits()  # the defaults on a launch of 96 tiles
        raster.autotune(scene, cam, poses, times, ws, torch.rand(4, 3, 64, 96, device="cuda"), cache_path=str(cache))
        line = json.loads(cache.read_text())
        for setting in ((128, 512, 52, 64), (128, 1024, 52, 64)):  # the second: the defaults' own values
            raster.set_tuning(128, 512, 52, 128)
            one_wave = bits()
            assert same_gradients(one_wave, quadrant) != []
            line.update(batch=setting[0], sort_cap=setting[1], compact=setting[2], bwd_batch=setting[3])
            cache.write_text(json.dumps(line) + "\n")
            t = raster.autotune(scene, cam, poses, times, ws, torch.rand(4, 3, 64, 96, device="cuda"),
                                cache_path=str(cache))
            assert raster.get_tuning() == t
            assert same_gradients(one_wave, bits()) == []
            two = bits(2)
            raster.set_tuning(256, 1024, 4, 256)
            raster.set_tuning(t["batch"], t["sort_cap"], t["compact"], t["bwd_batch"])
            assert same_gradients(one_wave, bits()) == [] and same_gradients(two, bits(2)) == []
    finally:
        raster.set_tuning(old["batch"], old["sort_cap"], old["compact"], old["bwd_batch"])
    assert same_gradients(quadrant, bits()) == []
