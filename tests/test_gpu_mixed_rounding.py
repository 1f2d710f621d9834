"""How often the mixed path rounds T_LR to FP32, seen through rotations of a dimer.

Each of 300 two-atom structures holds the same pair of carbon atoms (3.5 A apart, one atom per
local SCS) in another direction, so that the pair's FP32 coefficients are the same in all and
the ratio of the mixed energy to the FP64 energy moves with the rounding of the 3 x 3 block's
elements, of the Krylov vectors and of the products alone.  With c_2 only the energy is u_1's
norm, with c_4 only u_2's, one product further.  Its spread (standard deviation) over random
directions, from a NumPy model of the roundings (4,000 directions): u_1 from elements that were
formed in FP64 and rounded once 3.2e-8, from unrounded elements 1.2e-8, from s = sqrt(A) rhat
rounded before the elements are formed 8.3e-8; u_2 by products with elements rounded once
4.4e-8 .. 7.3e-8, by the lists' products with s 1.2e-7, with both from the rounded s 2.2e-7.
The limits lie between."""
import dataclasses

import numpy as np
import pytest

from workloads import SPECIES_TABLE
from tests.gpu_common import method_params

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=0.6, r_nbr=8.0, r_mbd1=8.0, r_mbd2=3.0)


@pytest.mark.parametrize("form,order,limit", [("dense", 2, 4.0e-8), ("dense", 4, 1.0e-7), ("sparse", 2, 4.0e-8),
                                              ("sparse", 4, 1.6e-7)])
def test_spread_over_rotations(form, order, limit):
    import torch
    from paper_2407_06409_amd import Context, compute_batch
    dev = torch.device("cuda:0")
    v = np.random.default_rng(17).normal(size=(300, 3))
    v *= 1.75 / np.linalg.norm(v, axis=1)[:, None]
    structs = [dict(pos=torch.tensor(np.array([x, -x]), device=dev), species=torch.ones(2, dtype=torch.int32, device=dev),
                    v_ratio=torch.full((2,), 0.8, dtype=torch.float64, device=dev), cell=None, pbc=(0, 0, 0),
                    cutoffs=CUT) for x in v]
    ctx = Context(0)
    ctx.set_mbd_product(form)
    c_n = [0.0] * order + [-1.0]
    e = {}
    for precision in ("fp64", "mixed"):
        print(f"{form} c_{order} {precision}", flush=True)
        prm = dataclasses.replace(method_params(n_max=order, precision=precision), c_n=c_n)
        out = compute_batch(structs, prm, SPECIES_TABLE, forces=False, ctx=ctx)
        e[precision] = np.array([o["energies"].cpu().numpy()[0] for o in out])
    assert np.ptp(e["fp64"]) < 1e-12 * abs(e["fp64"][0])
    spread = (e["mixed"] / e["fp64"]).std()
    print(f"  spread {spread:.2e}, limit {limit:.1e}", flush=True)
    assert spread < limit
