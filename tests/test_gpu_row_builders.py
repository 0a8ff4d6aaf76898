"""Neighbour rows at the edges of the builders, against the float64 oracle.

Boxes of four cells a side and of fewer along one vector, open boundaries, a
tilted box, stencils of more candidates than are staged at once, rows longer than a
candidate list, cells of more atoms than a block takes, a box that is mostly
empty, and a thin one whose rows hold periodic images: each alone (below
16,384 atoms a wave takes an atom) and repeated beyond that number (sixteen
lanes).  Rows are whole numbers and equal the oracle's.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth

pytestmark = pytest.mark.gpu

# atoms along each vector, spacing, box lengths (None: the grid's), tilt, periodic
CASES = {
    "four-cells": ((8, 8, 8), 2.4, None, 0.0, (1, 1, 1)),
    "three-cells": ((10, 8, 6), 2.4, None, 0.0, (1, 1, 1)),
    "open": ((9, 8, 7), 2.4, None, 0.0, (0, 1, 0)),
    "tilted": ((9, 8, 8), 2.5, None, 0.25, (1, 1, 1)),
    "dense": ((15, 15, 15), 1.4, None, 0.0, (1, 1, 1)),
    "crowd": ((9, 9, 9), 0.9, (40.0, 40.0, 40.0), 0.0, (1, 1, 1)),
    "sparse": ((8, 8, 8), 20.0, None, 0.0, (1, 1, 1)),
    "thin": ((3, 3, 40), 2.4, None, 0.1, (1, 1, 1)),
    "small": ((5, 5, 5), 2.2, None, 0.1, (1, 1, 0)),
}


def _cell(name):
    grid, a, lengths, tilt, pbc = CASES[name]
    rng = np.random.default_rng(len(name) + grid[2])
    L = np.array([g * a for g in grid] if lengths is None else lengths)
    box = np.diag(L) @ (np.eye(3) + tilt * np.triu(rng.uniform(-1, 1, (3, 3)), 1))
    at = np.stack(np.meshgrid(*[np.arange(g) + 0.5 for g in grid], indexing="ij"), -1).reshape(-1, 3) * a
    at += rng.uniform(-0.25 * a, 0.25 * a, at.shape)
    pos = (at / L) @ box
    return np.ascontiguousarray(pos[rng.permutation(len(pos))].T), box, pbc


def _rows(rows, pos, box, n):
    """Sorted (partner within the cell, displacement) of each row."""
    out = []
    for i, (j, shift) in rows:
        d = pos[:, j].T + shift @ box - pos[:, i]
        order = np.lexsort(np.rint(d * 1e5).astype(np.int64).T[::-1])
        out.append((j[order] % n, d[order]))
    return out


@pytest.mark.parametrize("name", CASES)
def test_rows_equal_the_oracle(name):
    pos, box, pbc = _cell(name)
    n = pos.shape[1]
    h = synth.hparams(1, 4.6, 3.7, 2, 2, 2, 2, 2, 0, 0, 4, 1)
    handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=1))
    copies = 16384 // n + 2
    axis = 1  # periodic in every case
    big = np.concatenate([pos + (c * box[axis])[:, None] for c in range(copies)], 1)
    long_box = box.copy()
    long_box[axis] *= copies
    for which, rc in ((0, 4.6), (1, 3.7)):
        ref = O.pairs(pos, box.reshape(9), rc, pbc)
        got = handle.neighbors(pos, box.reshape(9), which, pbc, cap=1024)
        want = _rows(enumerate(ref), pos, box, n)
        print(f"[rows] {name} {which}: longest {max(len(j) for j, _ in ref)}", flush=True)
        for (j, s), (jr, sr) in zip(got, ref):
            assert sorted(zip(j.tolist(), map(tuple, s.tolist()))) == sorted(zip(jr.tolist(), map(tuple, sr.tolist())))
        rows = handle.neighbors(big, long_box.reshape(9), which, pbc, cap=1024)
        assert [len(j) for j, _ in rows] == [len(j) for j, _ in ref] * copies
        some = [c * n + a for c in (0, copies // 2, copies - 1) for a in range(n)]
        for i, (j, d) in zip(some, _rows([(i, rows[i]) for i in some], big, long_box, n)):
            assert np.array_equal(j, want[i % n][0]) and np.abs(d - want[i % n][1]).max(initial=0.0) < 1e-8
    handle.close()


@pytest.mark.parametrize("name", [n for n in CASES if n not in ("crowd", "dense")])
@pytest.mark.parametrize("many", [False, True])
def test_rows_filtered_from_candidates_give_the_same_steps(name, many):
    """Rows filtered each step from candidates at r_c + skin against rows built
    anew: forces differ by at most twice the 1e-4 eV/A of the float32 path, so
    positions of mass 12 after 4 steps of 1 fs by at most
    2e-4 x 9.65e-3 / 12 x 4^2 / 2 < 2e-6 A."""
    pos, box, pbc = _cell(name)
    n = pos.shape[1]
    if many:
        copies = 16384 // n + 2
        pos = np.concatenate([pos + (c * box[1])[:, None] for c in range(copies)], 1)
        box = box * np.array([1, copies, 1])[:, None]
    h = synth.hparams(1, 4.6, 3.7, 2, 2, 2, 2, 2, 0, 0, 4, 1)
    vel = np.random.default_rng(5).normal(0, 2e-3, pos.shape)
    out = []
    for skin in (0.0, 0.6):
        handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=1), skin=skin)
        out.append(handle.md_run(pos, vel, np.zeros(pos.shape[1], np.int32), [12.0], box.reshape(9), 1.0, 4, 0, pbc)[0])
        handle.close()
    err = np.abs(out[0] - out[1]).max()
    print(f"[rows] {name} x{pos.shape[1] // n} with a skin: {err:.1e}", flush=True)
    assert np.isfinite(out[0]).all() and err < 2e-6


def test_rows_that_outgrow_their_capacity_during_a_run():
    """216 carbon atoms of a random model contract: their longest radial row passes the
    60 slots of the first capacity near step 460, in the middle of a chunk of
    steps, which is then evaluated on truncated rows and replayed on longer ones.
    A handle whose rows are long from the start gives the same bits."""
    h = synth.WORKLOADS["diamond216"]
    pos, types, box = synth.diamond216()
    m = np.array(synth.MASSES["diamond216"])
    vel = synth.maxwell_velocities(m[types], 300.0)
    out = []
    for grown in (False, True):
        handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=synth.SEED_WEIGHTS))
        if grown:
            handle.neighbors(pos * 0.6, box * 0.6, 0, cap=512)
        out.append(handle.md_run(pos, vel, types, m, box, 1.0, 520, 0))
        handle.close()
    assert max(len(j) for j, _ in O.pairs(out[0][0], box, h["rc_radial"])) > 60
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
