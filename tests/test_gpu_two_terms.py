"""n_max = 2 with forces (no column is left for the product that forms Tbar, which is then the
two-body radii's or the central atom's alone) in the dense form, through the C ABI, against the
oracle: FP64 within 1e-8 eV and 1e-8 eV/A, mixed precision within 1e-5 eV and 1e-4 eV/A."""
import numpy as np
import pytest

import oracle
from workloads import SPECIES_TABLE, frequency_grid
from workloads import configs as C
from tests.gpu_common import gpu_run, oracle_params

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=3.5, r_nbr=6.0, r_mbd1=4.0, r_mbd2=3.5)
TWO_BODY = dict(CUT, r_2b1=6.0, r_2b2=4.5)


@pytest.mark.parametrize("n,n_freq", [(17, 5), (40, 12)])
@pytest.mark.parametrize("cut", [CUT, TWO_BODY], ids=["mbd", "two_body"])
def test_two_terms_against_oracle(cut, n, n_freq):
    from paper_2407_06409_amd import Context
    st, grid = C.hcno_cluster(n, 700 + n), frequency_grid(n_freq)
    w = np.random.default_rng(n).uniform(0.5, 1.5, n)
    ctx = Context(0)
    ctx.set_mbd_product("dense")
    e, f = oracle.lmbd_energy_forces(st, oracle_params(cut, n_max=2, grid=grid), SPECIES_TABLE, weights=w)
    for precision, e_tol, f_tol in (("fp64", 1e-8, 1e-8), ("mixed", 1e-5, 1e-4)):
        print(f"{n} sites, {n_freq} nodes, n_max 2, {cut}, {precision}", flush=True)
        g = gpu_run(st, cut, n_max=2, weights=w, grid=grid, ctx=ctx, precision=precision)
        de, df = np.abs(g["energies"] - e).max(), np.abs(g["forces"] - f).max()
        print(f"  max |dE| {de:.3e} eV, max |dF| {df:.3e} eV/A (max |F| {np.abs(f).max():.3e})", flush=True)
        assert de < e_tol and df < f_tol
