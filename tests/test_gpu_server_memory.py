"""The server's memory budget holds: requests of several times the budget wait,
and what the card holds more while they run is the budget at most (and what
the allocator rounds up: 64 MiB)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_10046_amd import nep, synth

pytestmark = pytest.mark.gpu

H = synth.WORKLOADS["serve2"]


@pytest.mark.parametrize("dense", [False, True])
def test_server_stays_within_its_budget(dense):
    import torch
    budget = 1 << 30
    handle = nep.Handle(H, synth.random_params(O.num_params(H)))
    pos, types, box = synth.lattice("fcc", 13, 4.05, 0.05, 2)
    small = synth.lattice("fcc", 4, 3.4, 0.05, 2)   # longer rows than the others'
    handle.compute(*synth.lattice("fcc", 4, 4.05, 0.05, 2))
    before = torch.cuda.mem_get_info()[0]
    server = nep.Server(handle, budget, max_slots=64)
    tickets = [server.submit(pos, types, box, kind=nep.NEP_REQ_MD, vel=np.zeros_like(pos), n_steps=2,
                             masses=np.array(synth.MASSES["serve2"])) for _ in range(30)]
    if dense:
        tickets += [server.submit(*small) for _ in range(2)]
        tickets += [server.submit(pos, types, box) for _ in range(20)]
    used = 0
    first = None
    for t in tickets:
        got = server.poll(t, wait_ms=-1)
        used = max(used, before - torch.cuda.mem_get_info()[0])
        if len(got["U"]) == pos.shape[1] and "pos" not in got:
            first = got["U"] if first is None else first
            assert np.array_equal(got["U"], first)
    stats = server.stats()
    print(f"[server] {len(tickets)} x {pos.shape[1]} atoms, dense {dense}: {used / 2 ** 20:.0f} MiB, {stats}", flush=True)
    assert used <= budget + (64 << 20)
    assert stats["completed"] == len(tickets) and stats["mean_batch_requests"] > 2
    server.close()
    handle.close()
