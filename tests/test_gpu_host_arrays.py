"""Calls on host arrays: the staged copies (up to 8 MB) and the direct ones
beyond, every choice of outputs, and a handle that goes back and forth between
them, give the bits of the device call."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth

pytestmark = pytest.mark.gpu


def _compute(handle, pos, types, box, want):
    n = pos.shape[1]
    out = {k: np.full(s, 7.0) for k, s in dict(U=n, F=(3, n), W=(9, n), totals=10).items() if k in want}
    rc = nep.load().nep_compute(
        handle._h, n, nep._ptr(pos, C.c_double), nep._ptr(types, C.c_int32), nep._ptr(box, C.c_double), None,
        *(nep._ptr(out[k], C.c_double) if k in want else None for k in ("U", "F", "W", "totals")))
    assert rc == 0, nep.last_error(handle._h)
    return out


@pytest.mark.parametrize("cells", [4, 28])  # 256 atoms; 87,808: 9.1 MB of results, 30.9 MB of descriptors
def test_host_calls_equal_device_calls(cells):
    import torch
    h = synth.WORKLOADS["fcc131k"]
    handle = nep.Handle(h, synth.random_params(O.num_params(h), seed=2))
    pos, types, box = synth.lattice("fcc", cells, 4.05, 0.05, h["n_types"], 3)
    n = types.shape[0]
    ref = {k: torch.empty(s, dtype=torch.float64, device="cuda")
           for k, s in dict(U=(n,), F=(3, n), W=(9, n), totals=(10,)).items()}
    handle.compute_dev(torch.tensor(pos, device="cuda"), torch.tensor(types, device="cuda"), box, None,
                       ref["U"], ref["F"], ref["W"], ref["totals"])
    ref = {k: v.cpu().numpy() for k, v in ref.items()}
    box = np.ascontiguousarray(box, dtype=np.float64)
    for want in (("U", "F", "W", "totals"), ("F",), (), ("U", "totals"), ("W",), ("totals",), ("U", "F", "W", "totals")):
        for k, v in _compute(handle, pos, types, box, want).items():
            assert np.array_equal(v, ref[k]), (want, k)
    q = handle.descriptors(pos, types, box)
    idx = np.arange(0, n, max(n // 50, 1))
    print(f"[host arrays] {n} atoms, descriptors {q.shape}", flush=True)
    assert np.isfinite(q).all()
    assert np.array_equal(q, handle.descriptors(pos, types, box))
    if n < 1000:
        assert np.abs(q[idx] - O.descriptors(h, synth.random_params(O.num_params(h), seed=2), pos, types, box)[idx]).max() < 1e-4
    for k, v in _compute(handle, pos, types, box, ("U", "F", "W", "totals")).items():
        assert np.array_equal(v, ref[k]), k
    handle.close()
