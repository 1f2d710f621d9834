"""Sparse MBD products with more columns than a wavefront has lanes (3 n_freq / 2 in FP64 and
3 n_freq / 4 in mixed precision where they divide, else 3 n_freq): a second chunk of columns
with inactive lanes at its end, up to 32 nodes, and one wavefront per workgroup in the pair
pass at high n_max, through the C ABI, against the oracle (FP64 within 1e-8 eV and 1e-8 eV/A, mixed
precision within 1e-5 eV and 1e-4 eV/A)."""
import numpy as np
import pytest

import oracle
from workloads import SPECIES_TABLE, frequency_grid
from workloads import configs as C
from tests.gpu_common import gpu_run, oracle_params

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=3.5, r_nbr=9.0, r_mbd1=6.0, r_mbd2=3.0)


@pytest.mark.parametrize("n,n_freq,n_max,precision", [(20, 23, 4, "fp64"), (20, 22, 4, "mixed"), (20, 32, 12, "fp64"),
                                                      (31, 31, 5, "mixed"), (9, 25, 3, "fp64")])
def test_columns_beyond_one_wavefront(n, n_freq, n_max, precision):
    from paper_2407_06409_amd import Context
    st, grid = C.hcno_cluster(n, 800 + n), frequency_grid(n_freq)
    w = np.random.default_rng(n).uniform(0.5, 1.5, n)
    ctx = Context(0)
    ctx.set_mbd_product("sparse")
    print(f"{n} sites, {n_freq} nodes, n_max {n_max}, {precision}", flush=True)
    g = gpu_run(st, CUT, n_max=n_max, weights=w, grid=grid, ctx=ctx, precision=precision)
    e, f = oracle.lmbd_energy_forces(st, oracle_params(CUT, n_max=n_max, grid=grid), SPECIES_TABLE, weights=w)
    de, df = np.abs(g["energies"] - e).max(), np.abs(g["forces"] - f).max()
    print(f"  max |dE| {de:.3e} eV, max |dF| {df:.3e} eV/A (max |F| {np.abs(f).max():.3e})", flush=True)
    e_tol, f_tol = (1e-8, 1e-8) if precision == "fp64" else (1e-5, 1e-4)
    assert de < e_tol and df < f_tol
