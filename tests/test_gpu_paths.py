"""Kernels and dispatch branches at the sizes where they can go wrong, against the CPU oracle
(tests/parity.py: integers exactly, values within its stated tolerance)."""
import numpy as np
import pytest
import torch

from paper_2112_07221_amd import workloads as wl
from parity import Pair, run_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [1, 2])
def test_light_weight_lfu_where_the_select_gains_a_pass(cap):
    """A cap of 1 leaves rows of the batch that can be evicted unstamped (their trim has a kernel of its
    own for the tie count); from iteration 2048 the policy key has a second digit."""
    w = wl.WORKLOADS[1].scaled(batch=12, vocab=3_000, capacity=200, s=3, policy=wl.LFU_LIGHT)
    T = 2_070
    ids, grads, table = wl.IdStream(w).batches(T), wl.grad_pool(w), wl.table_init(w)
    p = Pair(w, table, lfu_cap=cap)
    try:
        ids_dev = torch.from_numpy(ids).to(p.dev)
        for t in range(T):
            p.lookup(ids[t], check_values=t % 64 == 0, ids_dev=ids_dev[t])
            p.update(ids[t], grads[t % len(grads)], ids_dev=ids_dev[t])
            if t % 256 == 0 or t >= 2_040:
                p.compare_state(values=False)
                p.compare_counters()
        p.flush_and_compare()
    finally:
        p.close()
