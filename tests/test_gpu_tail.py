"""Wide batches end on the narrow kernel where their last round of groups would
be nearly empty.  At the edges of that rule every gate's words are the
oracle's; the batch repeats eleven gates (prime, so that every place in a group
and on either side of the edge meets every gate).  The arithmetic is exact:
nothing but equality is accepted."""
import numpy as np
import pytest

import oracle
import paper_2005_01945_amd as F
import workloads

pytestmark = pytest.mark.gpu
GATES = 11


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    sk, ck = F.fhe_keygen(0)
    ops = workloads.gate_ops(190, GATES)
    c = [sk.encrypt_bits(workloads.bits(191 + k, GATES), nonce=8_000_000 + 1000 * k) for k in range(2)]
    want = oracle.Keys(0).bootstrap(ops, c[0], c[1], threads=8)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return F.Context(ck, 0), cus, ops, c, want


# whole compute units' worth of gates and gates beyond; a round is 8 per unit
@pytest.mark.parametrize("units, more",
                         [(4, 1), (5, 0), (5, 1), (8, 1), (9, 0), (9, 1), (10, 0), (10, 1), (12, 3), (13, 1)])
def test_tail_words(env, units, more):
    import torch
    ctx, cus, ops, c, want = env
    n = units * cus + more
    pick = np.arange(n) % GATES
    print(f"[gpu-test] {n} gates", flush=True)
    a, b = F.to_device(c[0][pick]), F.to_device(c[1][pick])
    out = torch.zeros_like(a)
    F.fhe_bootstrap_gate_batch(ctx, torch.from_numpy(ops[pick]).cuda(), a, b, out, n)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(F.to_host(out), want[pick])
