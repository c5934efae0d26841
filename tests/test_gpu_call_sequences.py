"""Calls that follow one another on the same workspace or change the
process-wide setting: each gives what it would give alone."""
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
