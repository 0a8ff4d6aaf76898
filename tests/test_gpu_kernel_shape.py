"""Quads of lanes per atom of the pair kernels: four below 16,384 atoms and one from
there on, by the atoms of each call; a batch keeps those of the first batch."""
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth

pytestmark = pytest.mark.gpu


def test_quads_on_both_sides_of_the_line():
    import torch
    h = synth.hparams(1, 4.6, 3.7, 2, 2, 2, 2, 2, 0, 0, 4, 1)
    handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=1))
    assert not any(handle.tuning().values())
    full = synth.lattice("fcc", 16, 4.05, 0.1, 1)     # 16,384 atoms
    for n, quads in ((16384, 1), (16383, 4), (300, 4), (16384, 1)):
        print(f"[shape] {n} atoms", flush=True)
        U = handle.compute(full[0][:, :n], full[1][:n], full[2])["U"]
        ref = O.evaluate_atoms(h, synth.random_params(O.num_params(h), seed=1), full[0][:, :n], full[1][:n], full[2],
                               list(range(0, n, 97)))["U"]
        assert abs(U[::97] - ref).max() <= 1e-5
        got = handle.tuning()
        assert [got["lanes_desc"], got["lanes_force"], got["lanes_gather"]] == [quads] * 3
    for first, quads in ((2, 4), (20, 1)):
        handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=1))
        for copies in (first, 22 - first):
            pos, types, boxes, offs = synth.concat_structures([synth.lattice("fcc", 6, 4.05, 0.1, 1)] * copies)
            handle.compute_batch(offs, torch.tensor(pos, device="cuda"), torch.tensor(types, device="cuda"), boxes, None,
                                 torch.empty(1, len(types), dtype=torch.float64, device="cuda"))
            assert handle.tuning(batch=True)["lanes_desc"] == quads
