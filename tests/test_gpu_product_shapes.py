"""The MBD products at the edges of their tiles, through the C ABI, against the oracle.

Dense form: 16-row strips and planes of 16 sites (n = 1, 16, 17, 33: 3n through strips with
remainders), one to more than three column tiles (3 n_freq = 9, 15, 36, 51), operands of the
adjoint whose K = n_max 3 n_freq is no multiple of 16, and n = 147 and 148 sites, where at 12
nodes in FP64 the products' operand is the last to fit in LDS and the first to stay in global
memory.  Sparse form: rows taken three at a time (n = 1, 2, 16, 65, 70: a short last triple,
up to and beyond 64 sites), an odd and an even number of columns (3 n_freq = 15, 36) and both
lengths of the moment loops (n_max up to 6 and beyond).  Every site sees the whole open
cluster; energies of sampled atoms and the forces of their weighted sum, FP64 within 1e-8 eV
and 1e-8 eV/A, mixed precision within 1e-5 eV and 1e-4 eV/A (Sec. III.B), as for every other
shape of the path."""
import numpy as np
import pytest

import oracle
from workloads import SPECIES_TABLE, frequency_grid
from workloads import configs as C
from tests.gpu_common import gpu_run, oracle_params

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=3.5, r_nbr=40.0, r_mbd1=40.0, r_mbd2=40.0)
CASES = [  # form, n, n_freq, n_max, precision, forces
    ("dense", 1, 12, 6, "fp64", True), ("dense", 16, 3, 4, "fp64", True), ("dense", 17, 5, 3, "mixed", True),
    ("dense", 33, 17, 7, "fp64", True), ("dense", 33, 5, 2, "fp64", True), ("dense", 147, 12, 4, "fp64", True),
    ("dense", 148, 12, 4, "fp64", True), ("dense", 119, 12, 4, "mixed", True),
    ("sparse", 1, 12, 6, "fp64", True), ("sparse", 2, 5, 2, "fp64", True), ("sparse", 16, 5, 3, "mixed", True),
    ("sparse", 65, 12, 6, "fp64", True), ("sparse", 70, 5, 8, "fp64", True), ("sparse", 70, 12, 5, "fp64", False),
]


@pytest.mark.parametrize("form,n,n_freq,n_max,precision,forces", CASES)
def test_product_shapes_against_oracle(form, n, n_freq, n_max, precision, forces):
    from paper_2407_06409_amd import Context
    st = C.hcno_cluster(n, 900 + n)
    grid = frequency_grid(n_freq)
    atoms = sorted({0, n // 2, n - 1})
    w = np.zeros(n)
    w[atoms] = [1.0, 0.5, -0.7][:len(atoms)]
    print(f"{form}: {n} sites, {n_freq} nodes, n_max {n_max}, {precision}", flush=True)
    ctx = Context(0)
    ctx.set_mbd_product(form)
    g = gpu_run(st, CUT, n_max=n_max, forces=forces, weights=w, grid=grid, ctx=ctx, precision=precision)
    e, f = oracle.lmbd_energy_forces(st, oracle_params(CUT, n_max=n_max, grid=grid), SPECIES_TABLE, weights=w,
                                     atoms=atoms)
    e_tol, f_tol = (1e-8, 1e-8) if precision == "fp64" else (1e-5, 1e-4)
    de = np.abs(g["energies"][atoms] - e[atoms]).max()
    print(f"  max |dE| {de:.3e} eV/atom", flush=True)
    assert de < e_tol
    if forces:
        df = np.abs(g["forces"] - f).max()
        print(f"  max |dF| {df:.3e} eV/A", flush=True)
        assert df < f_tol


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_operand_placement_does_not_change_results(precision):
    """A 33-atom cluster alone (the products' operand in LDS) and in one batch with a cluster of
    150 sites (operand of the whole launch in global memory): bitwise the same."""
    import torch
    from paper_2407_06409_amd import Context, compute_batch
    from tests.gpu_common import method_params
    dev = torch.device("cuda:0")

    def desc(n):
        st = C.hcno_cluster(n, 900 + n)
        return dict(pos=torch.as_tensor(st.pos, device=dev), species=torch.as_tensor(st.species, device=dev),
                    v_ratio=torch.as_tensor(st.nu, device=dev), cell=None, pbc=(0, 0, 0), cutoffs=CUT)

    print(f"33 sites alone and with 150, {precision}", flush=True)
    ctx = Context(0)
    ctx.set_mbd_product("dense")
    params = method_params(precision=precision)
    alone = compute_batch([desc(33)], params, SPECIES_TABLE, ctx=ctx)[0]
    batch = compute_batch([desc(33), desc(150)], params, SPECIES_TABLE, ctx=ctx)[0]
    for key in ("energies", "forces"):
        assert torch.equal(alone[key], batch[key]), key
