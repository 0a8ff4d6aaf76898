"""Memory of a population's branches: that of the batch, whatever else the handle
has run, grown with the batch and with the rows."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth
from tests.test_gpu_population_branches import _run

pytestmark = pytest.mark.gpu

H = synth.WORKLOADS["train3"]


def test_a_small_population_after_a_large_call_stays_small():
    import torch
    params = np.stack([synth.random_params(O.num_params(H), seed=60 + p) for p in range(4)])
    handle = nep.Handle(H, params[0])
    pos, types, box = synth.lattice("fcc", 40, 4.05, 0.05, 3)
    n = types.shape[0]
    small = synth.concat_structures(synth.random_structures(6, seed=5))
    want = _run(nep.Handle(H, params[0]), small, params)
    handle.compute_dev(torch.tensor(pos, device="cuda"), torch.tensor(types, device="cuda"), box, None,
                       torch.empty(n, dtype=torch.float64, device="cuda"))
    _run(handle, small, params[:1])  # the batch's own buffers: one branch
    before = torch.cuda.mem_get_info()[0]
    got = _run(handle, small, params)
    used = before - torch.cuda.mem_get_info()[0]
    print(f"[branches] {n} atoms, then 4 sets of {small[1].shape[0]}: {used / 2 ** 20:.0f} MiB", flush=True)
    # three branches of at most 8 KB an atom, and what the allocator rounds up to
    assert used < 3 * 8192 * small[1].shape[0] + (64 << 20)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    handle.close()


def test_growing_batches_and_rows_grow_the_branches():
    params = np.stack([synth.random_params(O.num_params(H), seed=60 + p) for p in range(4)])
    handle = nep.Handle(H, params[0])
    for count, seed in ((3, 1), (40, 2), (3, 1), (60, 3)):
        s = synth.concat_structures(synth.random_structures(count, seed=seed))
        want = _run(nep.Handle(H, params[0]), s, params)
        for a, b in zip(_run(handle, s, params), want):
            assert np.array_equal(a, b)
        print(f"[branches] {s[1].shape[0]} atoms", flush=True)
    pos, _, box = synth.lattice("fcc", 3, 2.6, 0.1, 1)  # longer rows from here on
    handle.neighbors(pos, box, 0, cap=512)
    for a, b in zip(_run(handle, s, params), want):
        assert np.array_equal(a, b)
    handle.close()
