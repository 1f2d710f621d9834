"""Atoms alone in their local SCS system (r_SCS below every distance): the system is 1 / abar times the
identity, so the polarisability at zero frequency is alpha0 nu.  FP64 within four roundings of one
ulp (1/abar, the pivot's reciprocal square root squared, the trace), 1e-15; mixed precision, FP32
solves with one refinement in FP64, within 2e-13, the square of an FP32 solve's few ulp; its rms is
6.9e-15 where a pivot's reciprocal square root is rounded once at its end and 9.6e-15 where it is
the product of two rounded factors (measured on these atoms): the limit lies between."""
import numpy as np
import pytest

from workloads import SPECIES_TABLE
from workloads import configs as C
from tests.gpu_common import gpu_run

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=0.6, r_nbr=3.0, r_mbd1=3.0, r_mbd2=3.0)


@pytest.mark.parametrize("precision,tol,rms_tol", [("fp64", 1e-15, 3e-16), ("mixed", 2e-13, 8e-15)])
def test_polarisability_of_lone_sites(precision, tol, rms_tol):
    st = C.hcno_box(1000, 77)
    print(f"{st.n} atoms, {precision}", flush=True)
    g = gpu_run(st, CUT, forces=False, precision=precision)
    exact = np.asarray(SPECIES_TABLE, dtype=np.float64).reshape(-1, 3)[st.species, 0] * st.nu
    err = np.abs(g["alpha_scs0"] / exact - 1.0)
    print(f"  relative error: rms {np.sqrt((err ** 2).mean()):.2e}, max {err.max():.2e}", flush=True)
    assert err.max() < tol and np.sqrt((err ** 2).mean()) < rms_tol
