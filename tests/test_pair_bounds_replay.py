"""Host replay of the pair kernels' addresses (no GPU): every global and LDS index
that k_descriptor, k_partial_forces and k_gather form, lane by lane, lies in
what the library allocates.

One and four quads of lanes per atom, structures alone (positions and images of
the row's entries, loaded up to two entries ahead; past the row the atom itself)
and in batches (stored displacements), and the gather's look-up through the
candidates of a filtered row.  Rows are the oracle's pairs in the library's
order.  Sizes that do not fill the last block, an atom without neighbours, and a
model of eight species whose sums and tables are the widest of their kind.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import synth
from tests.test_bounds_replay import Bounds, estimate_capacity, library_rows, pair_stride, round4, xcd_block

BLOCK = 256
H8 = synth.hparams(8, 4.6, 3.7, 3, 10, 4, 3, 2, 2, 1, 4, 1)


def _alone(n):
    """n atoms of a noisy crystal and one far from them, in an open box."""
    pos, types, _ = synth.lattice("fcc", 3, 4.05, 0.1, 8, seed=n)
    pos = np.concatenate([pos[:, :n] + 5.0, [[90.0], [90.0], [90.0]]], 1)
    return pos, np.append(types[:n], 7).astype(np.int32), (100.0 * np.eye(3)).reshape(9)


CASES = {
    "train3": (synth.WORKLOADS["train3"], synth.random_cell(40, 0.07, 0.2, 1.5, 3, np.random.default_rng(7))),
    "alloy": (synth.WORKLOADS["fcc131k"], synth.lattice("fcc", (3, 3, 2), 4.05, 0.1, 4, seed=2)),
    "species8": (H8, _alone(66)),
}


def _setup(name):
    h, (pos, types, box) = CASES[name]
    pos = np.asarray(pos)
    rows, rev = library_rows(pos, box, h["rc_radial"], h["rc_angular"])
    vol = abs(np.linalg.det(box.reshape(3, 3)))
    MR = max(estimate_capacity(h["rc_radial"], pos.shape[1] / vol), max(len(r[0]) for r in rows))
    nA, KA, L = h["n_max_angular"] + 1, h["basis_angular"] + 1, h["l_max_3b"]
    nd = O.num_descriptors(h)
    M = dict(T=h["n_types"], nR=h["n_max_radial"] + 1, KR=h["basis_radial"] + 1, nA=nA, KA=KA, L=L, ND=nd,
             NDp=(nd + 7) // 8 * 8, NT=(nA + 3) // 4, NBT=((L + 1) ** 2 + 2) // 4, MR=MR,
             many=L + int(h["l_max_4b"] >= 2) + int(h["l_max_5b"] >= 1))
    M["cA_pair"] = pair_stride(KA * round4(nA))
    return pos, types, box, rows, rev, h, M


def _lanes(N, per_atom, block=BLOCK):
    """(thread, atom, atom in range) of every thread of the grid, wave by wave."""
    nb = -(-N * per_atom // block)
    for blk in range(nb):
        first = xcd_block(blk, nb) * block
        for w in range(0, block, 64):
            yield [(w + l, min((first + w + l) // per_atom, N - 1), (first + w + l) // per_atom < N)
                   for l in range(64)]


def _walk(b, N, i, sub, nn, step, iters, j, types, batch):
    """(m, species) of the entries a lane visits, with the loads on the way."""
    def entry(m):
        e = m * N + i if m < nn else i
        if batch:
            b.touch("disp", e)
        else:
            b.touch("nl", e)
            b.touch("cd", e)

    def atom(m):
        k = j[m] if m < nn else i
        if not batch:
            for c in range(3):
                b.touch("pos", c * N + k)
            b.touch("types", k)
    entry(sub)
    entry(sub + step)
    atom(sub)
    for k in range(iters):
        m = sub + k * step
        atom(m + step)
        entry(m + 2 * step)
        yield m, (types[j[m]] if m < nn else 0 if batch else types[i])


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("Q", [1, 4])
@pytest.mark.parametrize("name", CASES)
def test_descriptor_and_partial_forces(name, Q, batch):
    pos, types, box, rows, _, h, M = _setup(name)
    N, T, KR, KA, NT, NBT = pos.shape[1], M["T"], M["KR"], M["KA"], M["NT"], M["NBT"]
    WR, W, KRp, atoms = round4(M["nR"]), 4 * NT, KR | 1, 64 // (4 * Q)
    tabR, tabA = T * T * KR * WR, T * T * M["cA_pair"]
    for force in (False, True):
        slots = T * KRp * (BLOCK // (4 * Q)) if force else 0
        b = Bounds(dict(nl=M["MR"] * N, cd=M["MR"] * N, disp=M["MR"] * N, pos=3 * N, types=N, q=N * M["NDp"],
                        fp=N * M["NDp"], sums=NT * NBT * 16 * N, P=M["MR"] * N, F=3 * N, sR=tabR, sA=tabA, At=slots))
        assert tabR % 4 == 0 and tabA % 4 == 0  # staged four floats at a time
        assert 4 * (tabR + tabA + slots) <= 64 * 1024
        stored = set()
        for wave in _lanes(N, 4 * Q):
            nn = {t: (len(rows[i][0]) if live else 0) for t, i, live in wave}
            na = {t: (rows[i][2] if live else 0) for t, i, live in wave}
            steps = max(-(-n // (4 * Q)) for n in nn.values())
            for t, i, live in wave:
                sub, s, lane, ti = t % (4 * Q), t % 4, t % 64, types[i]
                for u in range(NT):
                    for k in range(NBT):
                        if live or force:
                            b.touch("sums", (((u * NBT + k) * N + i) * 4 + s) * 4 + 3)
                at = (t // 64) * T * KRp * atoms + lane // (4 * Q)
                buf = "fp" if force else "q"
                if force or live:
                    for n in [k for k in range(M["nR"]) if force or k // 4 == s] + \
                             [M["nR"] + l * M["nA"] + 4 * u + s for l in range(M["many"]) for u in range(NT)
                              if 4 * u + s < M["nA"]]:
                        b.touch(buf, i * M["NDp"] + n)
                    b.touch(buf, i * M["NDp"] + (M["ND"] - 1 if force else M["NDp"] - 1))
                for k in range(T):
                    b.touch("sR", (ti * T + k) * KR * WR + (KR - 1) * WR + min(4 * s, WR - 4) + 3)
                    if force and k % (4 * Q) == sub:
                        b.touch("At", at + (k * KRp + KR - 1) * atoms)
                for m, tj in _walk(b, N, i, sub, nn[t], 4 * Q, steps, rows[i][0], types, batch):
                    b.touch("sA", (ti * T + tj) * M["cA_pair"] + (KA - 1) * W + W - 1)
                    if force:
                        b.touch("At", at + (tj * KRp + KR - 1) * atoms)
                        if m < nn[t]:
                            b.touch("P", i * M["MR"] + m)
                            assert (i, m) not in stored
                            stored.add((i, m))
                if live and sub < 3:
                    b.touch("F", sub * N + i)
                assert na[t] <= nn[t]
        b.check((name, Q, batch, force))
        assert not force or len(stored) == sum(len(r[0]) for r in rows)


@pytest.mark.parametrize("look_up", [False, True])
@pytest.mark.parametrize("G", [4, 16])
@pytest.mark.parametrize("name", CASES)
def test_gather(name, G, look_up):
    pos, types, box, rows, rev, h, M = _setup(name)
    N, MR = pos.shape[1], M["MR"]
    if look_up:  # rows filtered from candidates at r_c + 0.6 A, which every exact entry's position refers to
        cand = O.pairs(pos, box, h["rc_radial"] + 0.6)
        at = [{(int(j), *map(int, s)): k for k, (j, s) in enumerate(zip(*c))} for c in cand]
        MV = max(len(c[0]) for c in cand)
        fmap = -np.ones((MV, N), int)
        for i, (j, s, _) in enumerate(rows):
            for m, key in enumerate(zip(j.tolist(), s.tolist())):
                fmap[at[i][(key[0], *key[1])], i] = m
    b = Bounds(dict(nl=MR * N, rev=MR * N, cd=MR * N, disp=MR * N, pos=3 * N, P=MR * N, F=3 * N, W=9 * N,
                    fmap=(MV if look_up else 1) * N))
    for wave in _lanes(N, G):
        for t, i, live in wave:
            if not live:
                continue
            sub, (j, s, _) = t % G, rows[i]
            nn = len(j)

            def words(m):
                if m >= nn:
                    return 0, 0, None
                for buf in ("nl", "rev", "cd"):
                    b.touch(buf, m * N + i)
                if not look_up:
                    return j[m], rev[i][m], m
                return j[m], at[j[m]][(i, *(-s[m]).tolist())], m

            def partial(w):
                p = w[1]
                if look_up:
                    b.touch("fmap", p * N + w[0])
                    p = min(max(fmap[p, w[0]], 0), MR - 1)
                b.touch("P", w[0] * MR + p)
                if w[2] is not None:  # the entry that points back
                    back = rows[w[0]]
                    assert back[0][p] == i and np.array_equal(back[1][p], -s[w[2]])
            b.touch("disp", min(sub, max(nn - 1, 0)) * N + i)
            for m in [sub] + list(range(sub, nn, G)):
                for k in range(4):  # an entry and the three after it, past the row too
                    w = words(m + k * G)
                    partial(w)
                    for c in range(3):
                        b.touch("pos", c * N + w[0])
                if nn:
                    b.touch("disp", min(m + G, nn - 1) * N + i)
            for v in range(9):
                if v % G == sub:
                    b.touch("W", v * N + i)
            if sub < 3:
                b.touch("F", sub * N + i)
    b.check((name, G, look_up))
