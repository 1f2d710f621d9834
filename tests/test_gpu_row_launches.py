"""A batch whose largest neighbourhood gives every atom so many workgroups that one launch could
not count its work-items in 32 bits: a one-atom carbon cell with r_nbr = 42 A (about 31,000 sites)
and 6,720 atoms in small two-radius boxes.  Every structure's energies are bitwise those of a call
of its own kind alone."""
import numpy as np
import pytest

from workloads import SPECIES_TABLE
from workloads import configs as C
from tests.gpu_common import method_params

pytestmark = pytest.mark.gpu


def test_one_large_neighbourhood_among_many_atoms():
    import torch
    from paper_2407_06409_amd import Context, compute_batch
    dev = torch.device("cuda:0")

    def desc(st, **cut):
        return dict(pos=torch.as_tensor(st.pos, device=dev), species=torch.as_tensor(st.species, device=dev),
                    v_ratio=torch.as_tensor(st.nu, device=dev), cell=st.cell, pbc=tuple(int(x) for x in st.pbc),
                    cutoffs=cut)

    large = desc(C.carbon_box(1, 50), r_scs=4.0, r_nbr=42.0, r_mbd1=42.0, r_mbd2=3.0)
    small = [desc(C.carbon_box(64, 60 + i), r_scs=4.0, r_nbr=6.0, r_mbd1=4.0, r_mbd2=2.5) for i in range(3)]
    ctx, prm = Context(0), method_params(n_max=4)
    print("alone", flush=True)
    own = [o["energies"].cpu().numpy() for o in compute_batch(small, prm, SPECIES_TABLE, forces=False, ctx=ctx)]
    one = compute_batch([large], prm, SPECIES_TABLE, forces=False, ctx=ctx)[0]["energies"].cpu().numpy()
    print("one batch", flush=True)
    out = compute_batch([large] + small * 35, prm, SPECIES_TABLE, forces=False, ctx=ctx)
    assert np.array_equal(out[0]["energies"].cpu().numpy(), one)
    for i, o in enumerate(out[1:]):
        assert np.array_equal(o["energies"].cpu().numpy(), own[i % 3]), i
