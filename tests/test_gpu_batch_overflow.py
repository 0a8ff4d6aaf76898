"""Batches whose rows outgrow the capacity estimated from the mean density: a
cluster in a box that is mostly vacuum has up to 49 neighbours where 32 are
expected.  The call grows the rows, and everything that lies along them, and
tries again.  Results are the oracle's, and the bits of a handle whose rows
were long enough from the start, for a population, on reused rows and through
the server; with four quads of lanes per atom and, repeated beyond 16,384
atoms, with one."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth

pytestmark = pytest.mark.gpu

H = synth.hparams(2, 6.0, 5.0, 4, 4, 5, 5, 4, 2, 0, 16, 0)


def _clusters(seed=0):
    """Spheres of 30 to 50 atoms cut from crystals, in boxes of 20 to 26 A."""
    out = []
    for k, (kind, a, n) in enumerate((("fcc", 4.05, 50), ("bcc", 3.16, 44), ("diamond", 5.43, 30))):
        pos, types, box = synth.lattice(kind, 5, a, 0.1, 2, seed + k)
        pos -= box[0] / 2
        near = np.argsort((pos ** 2).sum(0))[:n]
        side = 20.0 + 3 * k
        out.append((np.ascontiguousarray(pos[:, near] + side / 2), types[near], (side * np.eye(3)).reshape(9)))
    return out


def _run(handle, s, params, reuse=False):
    import torch
    pos, types, boxes, offs = s
    n, P, S = types.shape[0], params.shape[0], len(offs) - 1
    out = [torch.full(k, np.nan, dtype=torch.float64, device="cuda")
           for k in ((P, n), (P, 3, n), (P, 9, n), (P, S, 10))]
    handle.compute_batch_dev(offs, torch.tensor(pos, device="cuda"), torch.tensor(types, device="cuda"), boxes,
                             torch.tensor(params, device="cuda"), *out, reuse_rows=reuse)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


def _grown(p):
    handle = nep.Handle(H, p)
    pos, _, box = synth.lattice("fcc", 3, 2.6, 0.1, 1)  # some 200 neighbours
    handle.neighbors(pos, box, 0, cap=512)
    return handle


@pytest.mark.parametrize("copies", [1, 140])
def test_rows_that_outgrow_their_capacity_in_a_batch(copies):
    structs = _clusters()
    params = np.stack([synth.random_params(O.num_params(H), seed=40 + k) for k in range(3)])
    ref = [[O.evaluate(H, p, *s) for s in structs] for p in params]
    longest = [max(len(j) for j, _ in O.pairs(s[0], s[2], 6.0)) for s in structs]
    print(f"[overflow] longest rows {longest}", flush=True)
    assert max(longest) > 32
    s = synth.concat_structures(structs * copies)
    handle, grown = nep.Handle(H, params[0]), _grown(params[0])
    want = _run(grown, s, params)
    for reuse in (False, True, False):
        got = _run(handle, s, params, reuse)
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
        for p in range(len(params)):
            at = 0
            for k in range(3 * copies):
                r = ref[p][k % 3]
                n = r["U"].shape[0]
                assert np.abs(got[0][p, at:at + n] - r["U"]).max() <= 1e-5
                assert np.abs(got[1][p, :, at:at + n] - r["F"]).max() <= 1e-4
                assert np.abs(got[2][p, :, at:at + n] - r["W"]).max() <= 1e-4
                at += n
        print(f"[overflow] {s[1].shape[0]} atoms, reuse {reuse}", flush=True)
    handle.close()
    grown.close()


def test_rows_that_outgrow_their_capacity_in_the_server():
    p = synth.random_params(O.num_params(H), seed=40)
    handle = nep.Handle(H, p)
    server = nep.Server(handle, 1 << 30, max_slots=8)
    structs = _clusters(5)
    tickets = [server.submit(*s, kind=nep.NEP_REQ_EVAL) for s in structs]
    for s, t in zip(structs, tickets):
        got, ref = server.poll(t, wait_ms=-1), O.evaluate(H, p, *s)
        print(f"[overflow] server, {s[1].shape[0]} atoms", flush=True)
        assert np.abs(got["U"] - ref["U"]).max() <= 1e-5 and np.abs(got["F"] - ref["F"]).max() <= 1e-4
    server.close()
    handle.close()
