"""Mixed precision: the gradient's pair terms are summed in FP64 by the lists' form.

The forces are linear in the seeds w_k, and a factor of a power of two is exact in every FP32
quantity that stays a normal number.  With seeds of 2^-120 the FP32 operands of Tbar (about
0.1 w_k) still are, with an error of 1e-45 / 1e-37 = 1e-8, while a pair's gradient, 1e-4 times
smaller at 5 A between the atoms, would be an FP32 denormal with an error of 1e-4.  One atom per
local SCS (r_SCS = 0.6 A), so that nothing but the MBD stage acts on the forces."""

import numpy as np
import pytest

from workloads import SPECIES_TABLE
from tests.gpu_common import method_params

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=0.6, r_nbr=20.0, r_mbd1=14.0, r_mbd2=6.0)
SCALE = 2.0 ** -120


def test_forces_are_linear_in_tiny_seeds():
    import torch
    from paper_2407_06409_amd import Context, compute
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(5)
    grid = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pos = 5.0 * grid + rng.uniform(-0.3, 0.3, size=grid.shape)
    n = len(pos)
    w = rng.choice([0.5, 1.0, 2.0], size=n)
    ctx = Context(0)
    ctx.set_mbd_product("sparse")
    f = []
    for scale in (1.0, SCALE):
        print(f"{n} atoms, seeds times {scale:.1e}", flush=True)
        out = compute(torch.as_tensor(pos, device=dev), torch.ones(n, dtype=torch.int32, device=dev),
                      torch.full((n,), 0.8, dtype=torch.float64, device=dev), cutoffs=CUT,
                      params=method_params(n_max=3, precision="mixed"), species_table=SPECIES_TABLE,
                      e_weight=torch.as_tensor(w * scale, device=dev), forces=True, ctx=ctx)
        f.append(out["forces"].cpu().numpy() / scale)
    err = np.abs(f[1] - f[0]).max() / np.abs(f[0]).max()
    print(f"  max |dF| / max |F| {err:.2e}", flush=True)
    assert err < 1e-6
