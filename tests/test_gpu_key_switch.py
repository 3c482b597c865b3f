"""Key switching on the int8 matrix cores against the oracle at the edges of its
gate tiles (32 or 64 gates) and of the shapes picked by batch width.  The sums
are exact integers, so the words must be equal."""
import numpy as np
import pytest

import oracle
import paper_2005_01945_amd as F
import workloads

pytestmark = pytest.mark.gpu
WIDEST = 577
SAMPLED = [0, 30, 31, 32, 63, 64, 127, 128, 255, 256, 511, 512, 575, 576]


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    sk, ck = F.fhe_keygen(0)
    ops = workloads.gate_ops(190, WIDEST)
    c0 = sk.encrypt_bits(workloads.bits(191, WIDEST), nonce=8_000_000)
    c1 = sk.encrypt_bits(workloads.bits(192, WIDEST), nonce=8_100_000)
    want = oracle.Keys(0).bootstrap(ops[SAMPLED], c0[SAMPLED], c1[SAMPLED], threads=8)
    return F.Context(ck, 0), torch.from_numpy(ops).cuda(), F.to_device(c0), F.to_device(c1), want


@pytest.mark.parametrize("count", [1, 31, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513, 577])
def test_tile_edges(env, count):
    import torch
    ctx, ops, a, b, want = env
    out = torch.zeros((count + 1, F.WORDS), dtype=torch.int32, device="cuda")
    F.fhe_bootstrap_gate_batch(ctx, ops, a, b, out, count)
    torch.cuda.synchronize()
    got = F.to_host(out)
    inside = [k for k, g in enumerate(SAMPLED) if g < count]
    np.testing.assert_array_equal(got[[SAMPLED[k] for k in inside]], want[inside])
    assert got[:count].any(axis=1).all() and not got[count].any()  # every gate written, nothing after the last
