"""Two forms of one kernel that a rule chooses between have to agree where the
rule may choose either, and keep what the general form accepts."""
import numpy as np
import pytest
import torch

from paper_1806_09907_amd import api

pytestmark = pytest.mark.gpu
DEV = "cuda"


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


# The squarings of a field that moves less than one voxel read their samples
# from LDS, the others from memory. One voxel of the second field moves two
# voxels, which sends its second squaring to memory; it reaches no sample more
# than a few voxels away, and there both squarings have the same inputs: the
# results must have the same bits.
@pytest.mark.parametrize("n", [(41, 27, 33), (34, 40, 21), (300, 37), (45, 70)])
def test_squaring_from_lds_and_from_memory_bitwise(n):
    d = len(n)
    rng = np.random.default_rng(11)
    th = rng.uniform(-1.6, 1.6, (d,) + tuple(reversed(n)))   # u_0 = theta / 4 in voxels
    far = th.copy()
    far[(0,) + (0,) * d] = 8.0
    for a in range(d):
        th[a] *= 2.0 / (n[a] - 1)
        far[a] *= 2.0 / (n[a] - 1)
    plan = api.Plan(api.Problem(n=n, transform=api.TF_DENSE, spacing=(1,) * d,
                                similarity=api.SIM_MSE, lambda_diff=0.0, diffeo_steps=2))
    print(f"case squaring forms {n}", flush=True)
    near_u = api.displacement(plan, gpu(th)).clone()
    far_u = api.displacement(plan, gpu(far)).clone()
    torch.cuda.synchronize()
    corner = (slice(None),) + (slice(0, 8),) * d
    assert not torch.equal(near_u[corner], far_u[corner])
    near_u[corner] = 0.0
    far_u[corner] = 0.0
    bad = (near_u != far_u).sum().item()
    assert bad == 0, f"{bad} of {near_u.numel()} differ"
