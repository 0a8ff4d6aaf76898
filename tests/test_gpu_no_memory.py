"""A call that finds no memory fails with NEP_E_OOM and leaves the handle fit for
the next, smaller one: rows of 60,000 slots for 330,000 atoms are more than the card
has (317 GB for the partial forces alone), those for 64 atoms are not."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth

pytestmark = pytest.mark.gpu


def test_a_smaller_call_after_one_that_found_no_memory():
    import torch
    h = synth.hparams(1, 4.6, 3.7, 2, 2, 2, 2, 2, 0, 0, 4, 1)
    handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=1), max_nb_radial=60000, max_nb_angular=60000)
    pos, types, box = synth.lattice("fcc", 3, 4.05, 0.1, 1)
    want = handle.compute(pos, types, box)
    assert 330000 * 60000 * 16 > torch.cuda.mem_get_info()[1]
    n = 330000
    big = torch.rand(3, n, dtype=torch.float64, device="cuda") * 300.0
    for call in range(2):
        print(f"[memory] call {call} for {n} atoms", flush=True)
        with pytest.raises(nep.NepError) as e:
            handle.compute_dev(big, torch.zeros(n, dtype=torch.int32, device="cuda"), (300.0 * np.eye(3)).reshape(9))
        assert e.value.code == nep.NEP_E_OOM
        got = handle.compute(pos, types, box)
        for k in ("U", "F", "W", "totals"):
            assert np.array_equal(got[k], want[k])
    handle.close()
