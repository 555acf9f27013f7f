"""A fused batch with more workgroups of one kind than a grid dimension holds
(2^32 threads): 4,097 pencils of one orbital at 4,096 shifts each, 2^24 + 4,096
workgroups of 256 threads per operation, go as several launches.  Every output
against the sum in closed form, sum_l Im(omega_l / (h - z_l s)): an error of at
most the 4,096 rounded additions, 4096 * 2^-53 < 1e-12 of the sum of moduli.
The systems share one workspace (its shifts and weights are the same for all).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_more_workgroups_than_one_grid_dimension_holds():
    import torch
    from paper_1405_0194_amd import binding as B
    nsys, P = 4097, 4096
    rng = np.random.default_rng(5)
    h, s = rng.uniform(-0.5, 0.5, nsys), rng.uniform(0.9, 1.1, nsys)
    z = rng.uniform(-0.6, 0.6, P) + 1j * rng.uniform(0.02, 0.4, P)
    w = (rng.standard_normal(P) + 1j * rng.standard_normal(P)) / P
    a = B.Analysis(1, np.array([0, 1]), np.array([0]))
    Hd, Sd = torch.from_numpy(h).cuda(), torch.from_numpy(s).cuda()
    per = P * a.info["bytes_per_shift"]
    L = torch.empty(nsys * per, dtype=torch.uint8, device="cuda")
    work = torch.empty(a.workspace_size(P), dtype=torch.uint8, device="cuda")
    print("case: batch of", nsys, "systems x", P, "shifts", flush=True)
    fb = B.FusedBatch([(a, Hd[i:i + 1], Sd[i:i + 1], P) for i in range(nsys)], nsets=1,
                      buffers=[(L[i * per:(i + 1) * per], work) for i in range(nsys)])
    print("launches", fb.launches, flush=True)
    assert fb.launches >= 4          # two operations, each in more than one launch
    fb.run([(z, w[None, :])] * nsys)
    torch.cuda.synchronize()
    got = torch.cat([o.reshape(-1) for o in fb.outputs()]).cpu().numpy()
    for i in list(range(0, nsys, 64)) + [1023, 1024, 1025, nsys - 1]:
        t = w / (h[i] - z * s[i])
        assert abs(got[i] - np.sum(t.imag)) <= 1e-12 * np.sum(np.abs(t)), i
