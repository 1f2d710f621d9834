"""The automatic choice of the MBD stage's form in the two-radius regime: clusters of up to 24 sites
per neighbourhood take the dense form, larger ones the sparse form, alone and in one batch (results
bitwise those of the form forced; the two forms differ in the last bits)."""
import numpy as np
import pytest

from workloads import SPECIES_TABLE
from workloads import configs as C
from tests.gpu_common import method_params

pytestmark = pytest.mark.gpu

CUT = dict(r_scs=4.0, r_nbr=40.0, r_mbd1=30.0, r_mbd2=6.0)   # every site sees the whole cluster


def test_automatic_form_by_size():
    import torch
    from paper_2407_06409_amd import Context, compute_batch
    dev = torch.device("cuda:0")

    def desc(n):
        st = C.hcno_cluster(n, 300 + n)
        return dict(pos=torch.as_tensor(st.pos, device=dev), species=torch.as_tensor(st.species, device=dev),
                    v_ratio=torch.as_tensor(st.nu, device=dev), cell=None, pbc=(0, 0, 0), cutoffs=CUT)

    def run(mode, sizes):
        ctx = Context(0)
        ctx.set_mbd_product(mode)
        out = compute_batch([desc(n) for n in sizes], method_params(), SPECIES_TABLE, ctx=ctx)
        return [(o["energies"].cpu().numpy(), o["forces"].cpu().numpy()) for o in out]

    same = lambda a, b: all(np.array_equal(x, y) for x, y in zip(a, b))  # noqa: E731
    batch = run("auto", (24, 25))
    for i, (n, form, other) in enumerate(((24, "dense", "sparse"), (25, "sparse", "dense"))):
        auto, forced, not_taken = run("auto", (n,))[0], run(form, (n,))[0], run(other, (n,))[0]
        assert not same(forced, not_taken)
        assert np.abs(forced[0] - not_taken[0]).max() < 1e-12 and np.abs(forced[1] - not_taken[1]).max() < 1e-12
        assert same(auto, forced), f"{n} sites"
        assert same(batch[i], forced), f"{n} sites in a batch"
