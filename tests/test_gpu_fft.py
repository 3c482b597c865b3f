"""The double-precision FFT kernels of blind rotation against the oracle, word
for word, where their work split can go wrong: groups of four gates that are
not full, more than one group, and every kind of gate input and output.  The
arithmetic is exact (the rounding bound is far below one half), so nothing but
equality is accepted."""
import numpy as np
import pytest

import oracle
import paper_2005_01945_amd as F
import workloads

pytestmark = pytest.mark.gpu
WIDEST = 1 << 31
GATES = 9


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    sk, ck = F.fhe_keygen(0)
    K = oracle.Keys(0)
    ops = workloads.gate_ops(170, GATES)
    c = [sk.encrypt_bits(workloads.bits(171 + k, GATES), nonce=7_000_000 + 1000 * k) for k in range(3)]
    return F.Context(ck, 0), K, ops, c, K.bootstrap(ops, c[0], c[1], threads=8)


def with_shape(ctx, shape, call):
    import torch
    try:
        F.fhe_ctx_set_launch_config(ctx, 1, WIDEST, shape)
        print(f"[gpu-test] shape {shape}", flush=True)
        call()
        torch.cuda.synchronize()
    finally:
        F.fhe_ctx_set_launch_config(ctx, 1, WIDEST, (1, 4, 1))


@pytest.mark.parametrize("shape", [(1, 4, 1), (2, 1, 1), (4, 1, 1)])
@pytest.mark.parametrize("count", [1, 2, 3, 4, 5, 8, 9])
def test_remainders(env, shape, count):
    import torch
    ctx, _, ops, c, want = env
    d_ops = torch.from_numpy(ops[:count].copy()).cuda()
    a, b = F.to_device(c[0][:count]), F.to_device(c[1][:count])
    out = torch.zeros_like(a)
    with_shape(ctx, shape, lambda: F.fhe_bootstrap_gate_batch(ctx, d_ops, a, b, out, count))
    np.testing.assert_array_equal(F.to_host(out), want[:count])


def test_group_kernel_inputs_and_outputs(env):
    """Three-input gates, a test vector, compound gates (two outputs) and an
    invalid code (all-zero output) in partly filled groups."""
    import torch
    ctx, K, _, c, _ = env
    n, shape = 6, (1, 4, 1)
    a, b, d = (F.to_device(x[:n]) for x in c)
    out, out1 = torch.zeros_like(a), torch.zeros_like(a)
    op3 = np.array([F.MAJ, F.XOR3] * 3, np.uint8)
    dev = lambda x: torch.from_numpy(np.asarray(x)).cuda()  # noqa: E731
    with_shape(ctx, shape, lambda: F.fhe_bootstrap_gate3_batch(ctx, dev(op3), a, b, d, out, n))
    np.testing.assert_array_equal(F.to_host(out), K.bootstrap3(op3, c[0][:n], c[1][:n], c[2][:n], threads=8))
    tv = workloads.rng(180).integers(0, 1 << 32, size=1024, dtype=np.uint32)
    with_shape(ctx, shape, lambda: F.fhe_bootstrap_lut_batch(ctx, F.to_device(tv), a, out, n))
    np.testing.assert_array_equal(F.to_host(out), K.bootstrap_lut(tv, c[0][:n], threads=8))
    o0, o1 = np.full(n, F.XOR, np.uint8), np.full(n, F.AND, np.uint8)
    with_shape(ctx, shape, lambda: F.fhe_bootstrap_compound_batch(ctx, dev(o0), dev(o1), a, b, out, out1, n))
    want = K.bootstrap_compound(np.stack([o0, o1], 1), c[0][:n], c[1][:n], threads=8)
    np.testing.assert_array_equal(F.to_host(out), want[:, 0])
    np.testing.assert_array_equal(F.to_host(out1), want[:, 1])
    ops = np.array([F.AND, 200, F.XOR, F.OR, F.NAND, F.MAJ], np.uint8)
    with_shape(ctx, shape, lambda: F.fhe_bootstrap_gate_batch(ctx, dev(ops), a, b, out, n))
    assert not F.to_host(out)[[1, 5]].any() and F.to_host(out)[[0, 2, 3, 4]].any(axis=1).all()
    with pytest.raises(F.FheError):
        F.fhe_ctx_check(ctx)


@pytest.mark.parametrize("shape", [(1, 4, 1), (2, 1, 1), (4, 1, 1)])
def test_valid_gates_beside_invalid_codes(env, shape):
    """Gates that share a group (or a launch) with invalid codes have the
    oracle's words."""
    import torch
    ctx, K, _, c, _ = env
    n, valid = 6, [0, 2, 3, 4]
    ops = np.array([F.AND, 200, F.XOR, F.OR, F.NAND, F.MAJ], np.uint8)
    a, b = F.to_device(c[0][:n]), F.to_device(c[1][:n])
    out = torch.full_like(a, 7)
    with_shape(ctx, shape, lambda: F.fhe_bootstrap_gate_batch(ctx, torch.from_numpy(ops).cuda(), a, b, out, n))
    got = F.to_host(out)
    np.testing.assert_array_equal(got[valid], K.bootstrap(ops[valid], c[0][valid], c[1][valid], threads=8))
    assert not got[[1, 5]].any()
    with pytest.raises(F.FheError):
        F.fhe_ctx_check(ctx)
