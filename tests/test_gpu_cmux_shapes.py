"""One CMux step on the kernel of every launch shape against the oracle, word for
word, on the data that the rounding bound of the FFT products is about: every
digit at an end of its range and both 16-bit halves of every key word at an end
of theirs, with signs that let one coefficient of the four-row sum reach 2^36 or
that put all of a transform's weight on one of its points.  Both arithmetics
are exact, so nothing but equality is accepted."""
import numpy as np
import pytest

import oracle
import paper_2005_01945_amd as F

N = 1024
KERNELS = [(1, 4, 1), (2, 1, 1), (4, 1, 1), (1, 4, 0)]
LOW, HIGH = -(1 << 15), (1 << 15) - 1
# accumulator words that a rotation by N (D = -2 acc) decomposes into these digits, twice
WORD_OF_DIGIT = {-512: 0xC0100400, 511: 0xC0100401}


def digits(D):
    x = (D.astype(np.int64) + 0x80200800) & 0xFFFFFFFF
    return [((x >> s) & 1023) - 512 for s in (22, 12)]


def word(hi, lo):
    """Key words of signed 16-bit halves."""
    return ((np.asarray(hi, np.int64) << 16) + np.asarray(lo, np.int64)).astype(np.uint32)


def acc_of(d):
    """Both accumulator polynomials from digits -512 or 511."""
    row = np.where(np.asarray(d) < 0, WORD_OF_DIGIT[-512], WORD_OF_DIGIT[511]).astype(np.uint32)
    return np.stack([row, row])


def key_of(hi, lo):
    return np.broadcast_to(word(hi, lo), (4, 2, N)).copy()


def one_coefficient(m):
    """Digits -512 and half words whose sum at coefficient m has all terms
    of one sign, each of the greatest magnitude."""
    k = np.where(np.arange(N) <= m, LOW, HIGH)
    return acc_of(np.full(N, -512)), k


def one_point(p):
    """Digits and half words with the signs of exp(i pi (2 p + 1) j / 1024), so
    that the transforms of both are greatest at the same root, and the product's
    coefficient 0 has all terms of one sign."""
    s = np.where(np.cos(np.pi * (2 * p + 1) * np.arange(N) / N) >= 0, 1, -1)
    k = np.empty(N, np.int64)
    k[0] = s[0]
    k[1:] = -s[:0:-1]
    return acc_of(s), np.where(k > 0, HIGH, LOW)


def cases():
    g = np.random.default_rng(36)
    for hi in (LOW, HIGH):
        for lo in (LOW, HIGH):
            yield f"constant {hi} {lo}", acc_of(np.full(N, -512)), key_of(hi, lo), N
    for m in (0, 31, 511, 512, 1000):
        acc, k = one_coefficient(m)
        yield f"coefficient {m}", acc, key_of(k, k), N
        yield f"coefficient {m}, halves of opposite sign", acc, key_of(-1 - k, k), N
    for p in (0, 1, 170, 511):
        acc, k = one_point(p)
        yield f"root {p}", acc, key_of(k, k), N
    for abar in (N, 1, 63, 64, 65, 1023, 1025, 2047):
        ends = g.choice([LOW, HIGH], size=(2, 4, 2, N))
        yield f"random ends, rotation {abar}", acc_of(g.choice([-1, 1], size=N)), word(ends[0], ends[1]), abar
        yield (f"random words, rotation {abar}", g.integers(0, 1 << 32, (2, N), dtype=np.uint64).astype(np.uint32),
               g.integers(0, 1 << 32, (4, 2, N), dtype=np.uint64).astype(np.uint32), abar)


def test_inputs_reach_the_ends():
    for d, w in WORD_OF_DIGIT.items():
        assert [int(x[0]) for x in digits(np.array([-2 * w & 0xFFFFFFFF], np.uint32))] == [d, d]
    for hi in (LOW, HIGH):
        for lo in (LOW, HIGH):  # the split of a key word: low half signed, the rest above it
            w = int(word(hi, lo))
            low = (w & 0xFFFF) - ((w & 0x8000) << 1)
            high = ((w - low) & 0xFFFFFFFF) >> 16
            assert (low, high - ((high & 0x8000) << 1)) == (lo, hi)
    for m in (0, 31, 511, 512, 1000, 1023):
        _, k = one_coefficient(m)
        terms = np.array([-512 * (int(k[m - j]) if j <= m else -int(k[N + m - j])) for j in range(N)])
        assert 4 * terms.sum() > (1 << 36) - (1 << 22) and (terms > 0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", KERNELS)
def test_cmux_at_the_ends(shape):
    for name, acc, bk, abar in cases():
        print(f"[gpu-test] cmux, shape {shape}: {name}", flush=True)
        np.testing.assert_array_equal(F.fhe_debug_cmux_shape(bk, abar, acc, shape), oracle.cmux(bk, abar, acc),
                                      err_msg=name)


def test_shapes_refused_on_the_host():
    """No call here reaches a GPU."""
    acc, bk = np.zeros((2, N), np.uint32), np.zeros((4, 2, N), np.uint32)
    for shape in [(1, 3, 0), (2, 2, 1), (4, 1, 0), (1, 4, 2), (3, 1, 1)]:
        with pytest.raises(F.FheError) as e:
            F.fhe_debug_cmux_shape(bk, 1, acc, shape)
        assert e.value.code == F.FHE_EINVAL
    for abar in (-1, 2 * N):
        with pytest.raises(F.FheError):
            F.fhe_debug_cmux_shape(bk, abar, acc, (1, 4, 1))
