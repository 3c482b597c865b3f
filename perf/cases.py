"""The work that programs have this framework do, as cases that can be timed.

A case is one pass through the public Python entry points: a gate batch, a
programmable-bootstrapping batch, an integer circuit, or a burst of jobs
through the server.  `listed()` names the fixed ones, `draw(rng)` gives others
of the same ranges, `prepare` makes what a program holds before the call (keys
on the GPU, encrypted inputs, output buffers), `run` makes the call and
`work` states the least bytes and operations of it.

Every output is a tensor of ciphertext words (int32 views of uint32), so
results compare word for word and there is no 64-bit value to be near.
"""
import functools

import numpy as np
import torch

import paper_2005_01945_amd as F

WORDS = F.WORDS  # 501 words per LWE sample
RING = 1024
LWE_N = 500

# Circuit entry points: (call, kind of fhe_circuit_shape).  The matrix product
# by vector has rows and cols; the others run `count` operand pairs.
CIRCUITS = {
    "add": (F.fhe_add, "add"),
    "add_fa": (F.fhe_add_fa, "add_fa"),
    "add_compound": (F.fhe_add_compound, "add_compound"),
    "add_numberwise": (F.fhe_add_numberwise, "add_numberwise"),
    "mul": (F.fhe_mul, "mul"),
    "mul_tree": (F.fhe_mul_tree, "mul_tree"),
    "mul_karatsuba": (F.fhe_mul_karatsuba, "karatsuba"),
    "matvec": (F.fhe_matvec, "matvec"),
}

# The job mix of a served burst: kind, integer width, rows, cols, share.
JOBS = [("gate", 1, 0, 0), ("add", 16, 0, 0), ("gate", 1, 0, 0), ("mul_tree", 8, 0, 0), ("gate", 1, 0, 0),
        ("add", 32, 0, 0), ("matvec", 4, 3, 2)]
JOB_KIND = {"gate": F.FHE_JOB_GATE, "add": F.FHE_JOB_ADD, "mul_tree": F.FHE_JOB_MUL_TREE,
            "matvec": F.FHE_JOB_MATVEC}


def listed():
    return [
        # one gate, waited for: an interactive program, and the baseline of
        # every batched figure
        {"name": "plain_gate", "path": "plain", "count": 1},
        # a handful of gates of mixed codes: a narrow level of a program that
        # drives the gates itself
        {"name": "gates_37", "path": "gates", "count": 37},
        # the batch of 1,024 gates that gate throughput is usually quoted on
        {"name": "gates_1024", "path": "gates", "count": 1024},
        # a wide ragged level, eight rounds of the chip and one gate
        {"name": "gates_16385", "path": "gates", "count": 16385},
        # the allocation-free entry, as called from a captured serving loop
        {"name": "noalloc_2500", "path": "noalloc", "count": 2500},
        # XOR and AND of the same bits (half adders), one rotation each
        {"name": "compound_777", "path": "compound", "count": 777},
        # majority and parity (full adders), an odd narrow batch
        {"name": "gate3_300", "path": "gate3", "count": 300},
        # a lookup table on encrypted messages
        {"name": "lut_5000", "path": "lut", "count": 5000},
        # 1,024 additions of 16-bit integers at once: a wide first level, then
        # a long carry chain of 2,048-gate levels; the largest case
        {"name": "add16_x1024", "path": "add", "width": 16, "count": 1024},
        # the latency of one 32-bit product: 62 levels, most of them narrow
        {"name": "mul_tree32_x1", "path": "mul_tree", "width": 32, "count": 1},
        # an 8-bit matrix-vector product as it is served
        {"name": "matvec_8x8_w8", "path": "matvec", "width": 8, "rows": 8, "cols": 8, "count": 1},
        # a burst of small mixed jobs through the continuous-batching server
        {"name": "serve_35", "path": "serve", "jobs": 35},
    ]


def _gates(case):
    """Bootstraps of one pass."""
    p = case["path"]
    if p == "serve":
        return sum(_gates({"path": k if k != "gate" else "gates", "width": w, "rows": r, "cols": c, "count": 1})
                   for k, w, r, c in _job_list(case))
    if p in CIRCUITS:
        g = F.fhe_circuit_shape(CIRCUITS[p][1], case["width"], case.get("rows", 0), case.get("cols", 0))[0]
        return g * case["count"]
    return case["count"]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    limit = _gates({"path": "add", "width": 16, "count": 1024})
    while True:
        p = rng.choice(["plain", "gates", "gates", "noalloc", "compound", "gate3", "lut", "circuit", "circuit",
                        "matvec", "serve"])
        if p == "plain":
            # one call per gate leaves nothing to vary but how many are made
            case = {"path": p, "count": _log_int(rng, 1, 60)}
        elif p == "gates":
            case = {"path": p, "count": _log_int(rng, 1, 16385)}
        elif p in ("noalloc", "compound", "gate3", "lut"):
            case = {"path": p, "count": _log_int(rng, 1, {"noalloc": 4096, "lut": 5000}.get(p, 4000))}
        elif p == "circuit":
            c = rng.choice(["add", "add_fa", "add_compound", "add_numberwise", "mul", "mul_tree", "mul_karatsuba"])
            case = {"path": c, "width": rng.randint(2, 32), "count": _log_int(rng, 1, 1024)}
        elif p == "matvec":
            case = {"path": p, "width": rng.randint(2, 16), "rows": rng.randint(1, 8), "cols": rng.randint(1, 8),
                    "count": 1}
        else:
            case = {"path": p, "jobs": rng.randint(1, 60)}
        # the widest circuits of the ranges hold far more gates than the
        # largest listed case; the long ones take a launch per level
        if _gates(case) <= limit // 2 and _levels(case) <= 80:
            return case


def _levels(case):
    if case["path"] in CIRCUITS:
        return F.fhe_circuit_shape(CIRCUITS[case["path"]][1], case["width"], case.get("rows", 0),
                                   case.get("cols", 0))[1]
    return case["count"] if case["path"] == "plain" else 1


@functools.lru_cache(maxsize=2)
def _keys(seed):
    return F.fhe_keygen(seed)


def _job_list(case):
    return [JOBS[k % len(JOBS)] for k in range(case["jobs"])]


def _uints(g, count, width):
    return g.integers(0, 1 << width, size=count, dtype=np.uint64)


def prepare(case, seed):
    sk, ck = _keys(seed)
    g = np.random.Generator(np.random.PCG64(seed + 1))
    ctx = F.Context(ck, 0)
    st = {"ctx": ctx, "case": dict(case)}
    nonce = [1 << 20]

    def bits(count):
        nonce[0] += count
        return F.to_device(sk.encrypt_bits(g.integers(0, 2, size=count, dtype=np.uint8), nonce=nonce[0] - count))

    def ints(count, width):
        nonce[0] += count * width
        return F.to_device(sk.encrypt_uint(_uints(g, count, width), width, nonce=nonce[0] - count * width))

    p = case["path"]
    if p == "plain":
        n = case["count"]
        st["ops"] = [int(k) for k in g.integers(0, 10, size=n)]
        a, b = bits(n), bits(n)
        out = F.empty_samples((n,))
        st["a"], st["b"] = [a[k] for k in range(n)], [b[k] for k in range(n)]
        st["rows"], st["out"] = [out[k] for k in range(n)], out
    elif p in ("gates", "noalloc"):
        n = case["count"]
        st["ops"] = torch.from_numpy(g.integers(0, 10, size=n, dtype=np.uint8)).cuda()
        st["a"], st["b"], st["out"] = bits(n), bits(n), F.empty_samples((n,))
    elif p == "gate3":
        n = case["count"]
        st["ops"] = torch.from_numpy(g.choice(np.array([F.MAJ, F.XOR3], np.uint8), size=n)).cuda()
        st["a"], st["b"], st["c"], st["out"] = bits(n), bits(n), bits(n), F.empty_samples((n,))
    elif p == "compound":
        n = case["count"]
        codes = np.array([F.XOR, F.AND], np.uint8)  # half adders
        st["ops0"] = torch.from_numpy(np.full(n, codes[0], np.uint8)).cuda()
        st["ops1"] = torch.from_numpy(np.full(n, codes[1], np.uint8)).cuda()
        st["a"], st["b"] = bits(n), bits(n)
        st["out0"], st["out1"] = F.empty_samples((n,)), F.empty_samples((n,))
    elif p == "lut":
        n = case["count"]
        # a table of 16 encrypted values over half the torus, as a program
        # builds it: 64 equal coefficients per entry
        table = g.integers(0, 16, size=16, dtype=np.uint32) << np.uint32(27)
        st["tv"] = F.to_device(np.repeat(table, RING // 16).astype(np.uint32))
        st["a"], st["out"] = bits(n), F.empty_samples((n,))
    elif p == "matvec":
        r, c, w = case["rows"], case["cols"], case["width"]
        st["a"], st["b"] = ints(r * c, w), ints(c, w)
        st["out"] = F.empty_samples((r, w))
    elif p == "serve":
        st["jobs"] = []
        for kind, w, r, c in _job_list(case):
            na, nb, no = (r * c, c, r) if kind == "matvec" else (1, 1, 1)
            st["jobs"].append((JOB_KIND[kind], int(g.integers(0, 10)), w, r, c, ints(na, w), ints(nb, w),
                               F.empty_samples((no, w))))
        torch.cuda.synchronize()  # a job's inputs are complete before it is submitted
        st["server"] = F.Server(ctx, 256 << 20)
    else:
        n, w = case["count"], case["width"]
        st["a"], st["b"] = ints(n, w), ints(n, w)
        st["out"] = F.empty_samples((n, 2 * w if p == "mul_karatsuba" else w))
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    p = case["path"]
    if p == "plain":
        for op, a, b, o in zip(st["ops"], st["a"], st["b"], st["rows"]):
            F.fhe_bootstrap_gate_plain(ctx, op, a, b, o)
        return st["out"]
    if p == "gates":
        F.fhe_bootstrap_gate_batch(ctx, st["ops"], st["a"], st["b"], st["out"])
        return st["out"]
    if p == "noalloc":
        F.fhe_bootstrap_gate_batch_noalloc(ctx, st["ops"], st["a"], st["b"], st["out"], case["count"])
        return st["out"]
    if p == "gate3":
        F.fhe_bootstrap_gate3_batch(ctx, st["ops"], st["a"], st["b"], st["c"], st["out"], case["count"])
        return st["out"]
    if p == "compound":
        F.fhe_bootstrap_compound_batch(ctx, st["ops0"], st["ops1"], st["a"], st["b"], st["out0"], st["out1"],
                                       case["count"])
        return [st["out0"], st["out1"]]
    if p == "lut":
        F.fhe_bootstrap_lut_batch(ctx, st["tv"], st["a"], st["out"], case["count"])
        return st["out"]
    if p == "matvec":
        F.fhe_matvec(ctx, st["a"], st["b"], st["out"], case["rows"], case["cols"], case["width"])
        return st["out"]
    if p == "serve":
        srv = st["server"]
        tickets = [F.fhe_serve_submit(srv, kind, a, b, out, op=op, width=w, rows=r, cols=c)
                   for kind, op, w, r, c, a, b, out in st["jobs"]]
        for t in tickets:
            F.fhe_serve_wait(srv, t)
        return [j[-1] for j in st["jobs"]]
    CIRCUITS[p][0](ctx, st["a"], st["b"], st["out"], case["count"], case["width"])
    return st["out"]


def _samples(case):
    """Ciphertexts read and written by one pass."""
    p = case["path"]
    if p == "serve":
        return sum(2 if k == "gate" else 3 * w if k != "matvec" else (r * c + c + r) * w
                   for k, w, r, c in _job_list(case))
    if p == "matvec":
        r, c = case["rows"], case["cols"]
        return (r * c + c + r) * case["width"]
    if p in CIRCUITS:
        return case["count"] * case["width"] * (4 if p == "mul_karatsuba" else 3)
    return case["count"] * {"lut": 2, "gate3": 4, "compound": 4}.get(p, 3)


def work(case):
    """Bytes: both keys (bootstrapping 500 x 8 polynomials of 1,024 words, the
    24,576 key-switching rows) and the samples once.  Operations per
    bootstrap: 500 external products, each four forward and two inverse
    transforms of 1,024 points (512-point complex form: 9 x 256 butterflies
    of ten operations) and 8 x 512 complex multiply-adds; then the 6,144
    expected key-switching rows of 501 words."""
    keys = LWE_N * 8 * RING * 4 + RING * 8 * 3 * WORDS * 4
    per_gate = LWE_N * (6 * 9 * 256 * 10 + 8 * 512 * 8) + 6144 * WORDS
    rows = 2 if case["path"] in ("compound", "add_compound") else 1
    extra = (rows - 1) * 6144 * WORDS
    gates = _gates(case)
    return {"bytes": keys + _samples(case) * WORDS * 4, "flops": gates * (per_gate + extra)}


def exact(case, seed):
    """Ciphertext words are whole numbers: equal or not, with nothing to be near."""
    return None
