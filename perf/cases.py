"""The work that users of this library have it do, as cases that can be timed and compared.

A fixed binary or ternary weight matrix is indexed once; activation vectors arrive later and are multiplied with the
index (include/rsr.h).  What varies in earnest: the matrix (from 1024 x 1024 to 32768 x 32768, binary or ternary,
uniform, sparse or with correlated rows), the block width k (near the one the paper's cost formula gives), the number of
vectors per call (one in decoding, up to sixteen when several sequences decode together), the activation type (float or
int8), and whether products go out one by one or several in a launch.  Building the index of a matrix that sits in device memory
is the other direction: it is what a program pays when it loads weights.

Matrices and activations are random, with the value laws of the benchmark configurations (workloads/configs.py).
"""
import math
import random
import weakref

import torch

import paper_2411_06360_amd as rsr

# Transformer block of configuration 4: model width 2560, feed-forward width 6912, 1.58-bit weights, k = 10.
BLOCK = {"q": (2560, 2560), "k": (2560, 2560), "v": (2560, 2560), "o": (2560, 2560), "gate": (2560, 6912), "up": (2560, 6912), "down": (6912, 2560)}
STAGES = {"qkv": (2560, 7680), "o": (2560, 2560), "gate_up": (2560, 13824), "down": (6912, 2560)}


def listed():
    return [
        # configuration 1: the smallest product of the benchmark; what a call costs
        {"name": "binary_1k_i8", "what": "product", "kind": "binary", "rows": 1024, "cols": 1024, "k": 8, "batch": 1, "dtype": "i8"},
        # configuration 2: an ordinary ternary layer, one vector
        {"name": "ternary_4k_f32", "what": "product", "kind": "ternary", "zeros": 1 / 3, "rows": 4096, "cols": 4096, "k": 10, "batch": 1, "dtype": "f32"},
        # configuration 3, the headline: one float vector, and eight (float and int8)
        {"name": "binary_16k_f32", "what": "product", "kind": "binary", "rows": 16384, "cols": 16384, "k": 12, "batch": 1, "dtype": "f32"},
        {"name": "binary_16k_f32_b8", "what": "product", "kind": "binary", "rows": 16384, "cols": 16384, "k": 12, "batch": 8, "dtype": "f32"},
        {"name": "binary_16k_i8_b8", "what": "product", "kind": "binary", "rows": 16384, "cols": 16384, "k": 12, "batch": 8, "dtype": "i8"},
        # configuration 4: one decode step of a transformer block.  One sequence: q/k/v and gate/up, which read the same
        # activations, go out as one launch each; the int8 activations of a BitLinear layer; sixteen sequences: q/k/v and
        # gate/up are one index each
        {"name": "block_f32", "what": "block", "zeros": 0.5, "k": 10, "batch": 1, "dtype": "f32"},
        {"name": "block_i8", "what": "block", "zeros": 0.5, "k": 10, "batch": 1, "dtype": "i8"},
        {"name": "block_f32_b16", "what": "stages", "zeros": 0.5, "k": 10, "batch": 16, "dtype": "f32"},
        # configuration 5: the largest, rows correlated through 64 prototypes (skewed segment lengths), four vectors
        {"name": "ternary_32k_f32_b4", "what": "product", "kind": "correlated", "zeros": 0.6, "rows": 32768, "cols": 32768, "k": 13, "batch": 4, "dtype": "f32"},
        # nothing divides anything: odd row and column counts, a narrow last block, an odd batch of int8 vectors
        {"name": "ragged_i8_b5", "what": "product", "kind": "ternary", "zeros": 1 / 3, "rows": 5003, "cols": 3001, "k": 11, "batch": 5, "dtype": "i8"},
        # a matrix with four bits per entry as weighted binary planes
        {"name": "fourbit_2k_f32", "what": "qbit", "bits": 4, "rows": 2048, "cols": 2048, "k": 9, "batch": 1, "dtype": "f32"},
        # weights arrive on the device: index them, take one product, let the index go
        {"name": "build_4k", "what": "build", "kind": "ternary", "zeros": 1 / 3, "rows": 4096, "cols": 4096, "k": 10, "batch": 1, "dtype": "f32"},
    ]


def _between(rng, low, high):
    """A whole number between low and high, spread over its logarithm; round numbers come up too."""
    x = math.exp(rng.uniform(math.log(low), math.log(high)))
    step = rng.choice([1, 1, 8, 64, 256])
    return int(min(high, max(low, round(x / step) * step)))


def _near_best_k(rng, rows):
    """Block widths that are used: around the minimum of the paper's cost (rows + 2^k) / k, within 8 .. 13."""
    best = min(range(8, 14), key=lambda k: (rows + 2**k) / k)
    return min(13, max(8, best + rng.choice([-1, 0, 0, 1])))


def draw(rng):
    what = rng.choice(["product"] * 7 + ["block", "stages", "qbit", "build"])
    dtype = rng.choice(["f32", "f32", "i8"])
    if what in ("block", "stages"):
        return {"what": what, "zeros": round(rng.uniform(0.3, 0.65), 3), "k": rng.choice([9, 10, 11]), "batch": rng.choice([1, 2, 3, 4, 7, 12, 16]), "dtype": dtype}
    if what == "qbit":
        rows, cols = _between(rng, 1024, 3000), _between(rng, 1024, 3000)
        return {"what": what, "bits": rng.choice([2, 3, 4]), "rows": rows, "cols": cols, "k": _near_best_k(rng, rows), "batch": rng.choice([1, 2, 4]), "dtype": dtype}
    most = 8192 if what == "build" else 32768
    rows, cols = _between(rng, 1024, most), _between(rng, 1024, most)
    kind = rng.choice(["binary", "ternary", "ternary", "correlated"])
    case = {"what": what, "kind": kind, "rows": rows, "cols": cols, "k": _near_best_k(rng, rows), "dtype": dtype}
    if kind != "binary":
        case["zeros"] = round(rng.uniform(0.3, 0.65), 3)
    case["batch"] = 1 if what == "build" else max(1, min(rng.choice([1, 1, 2, 3, 4, 5, 8, 11, 16]), 4 * 32768 * 32768 // (rows * cols)))
    return case


# ---- inputs, made on the device from the seed alone ------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _law(u, kind, zeros):
    """Entries by their law from uniform numbers in [0, 1)."""
    if kind == "binary":
        return (u < 0.5).to(torch.int8)
    side = (1.0 - zeros) / 2.0
    return (u < side).to(torch.int8) - (u >= 1.0 - side).to(torch.int8)


def _matrix(g, kind, rows, cols, zeros=0.0):
    A = torch.empty((rows, cols), dtype=torch.int8, device="cuda")
    step = max(1, (1 << 26) // cols)
    if kind == "correlated":  # every row is one of 64 prototype rows with 5 % of its entries drawn anew
        prototypes = _law(torch.rand((64, cols), generator=g, device="cuda"), kind, zeros)
        which = torch.randint(0, 64, (rows,), generator=g, device="cuda")
    for r in range(0, rows, step):
        n = min(step, rows - r)
        part = _law(torch.rand((n, cols), generator=g, device="cuda"), kind, zeros)
        if kind == "correlated":
            part = torch.where(torch.rand((n, cols), generator=g, device="cuda") < 0.05, part, prototypes[which[r:r + n]])
        A[r:r + n] = part
    return A


def _vectors(g, batch, rows, dtype):
    if dtype == "i8":
        return torch.randint(-127, 128, (batch, rows), generator=g, device="cuda", dtype=torch.int8)
    return torch.randn((batch, rows), generator=g, device="cuda", dtype=torch.float32)


def _result(batch, cols, dtype):
    return torch.zeros((batch, cols), dtype=torch.int32 if dtype == "i8" else torch.float32, device="cuda")


class _Held:
    """Indexes of a state: given back when the state goes."""

    def __init__(self, destroy):
        self.handles = []
        weakref.finalize(self, _Held.release, self.handles, destroy)

    @staticmethod
    def release(handles, destroy):
        torch.cuda.synchronize()
        for h in handles:
            destroy(h)

    def add(self, h):
        self.handles.append(h)
        return h


def _index(A, k):
    torch.cuda.synchronize()  # the builder works on the default stream
    return rsr.rsr_preprocess_device(A, A.shape[0], A.shape[1], k)


def prepare(case, seed):
    g = _generator(seed)
    what, batch, dtype = case["what"], case["batch"], case["dtype"]
    s = {"what": what, "batch": batch, "dtype": dtype, "stream": torch.cuda.current_stream().cuda_stream}
    if what == "product":
        A = _matrix(g, case["kind"], case["rows"], case["cols"], case.get("zeros", 0.0))
        s["held"] = _Held(rsr.rsr_destroy)
        s["h"] = s["held"].add(_index(A, case["k"]))
        s["v"], s["out"] = _vectors(g, batch, case["rows"], dtype), _result(batch, case["cols"], dtype)
    elif what in ("block", "stages"):
        s["held"] = _Held(rsr.rsr_destroy)
        x, a, h = _vectors(g, batch, 2560, dtype), _vectors(g, batch, 2560, dtype), _vectors(g, batch, 6912, dtype)
        y = _vectors(g, batch, 2560, dtype)
        reads = {"q": x, "k": x, "v": x, "qkv": x, "o": a, "gate": y, "up": y, "gate_up": y, "down": h}
        for name, (rows, cols) in (BLOCK if what == "block" else STAGES).items():
            A = _matrix(g, "ternary", rows, cols, case["zeros"])
            s[name] = (s["held"].add(_index(A, case["k"])), reads[name], _result(batch, cols, dtype))
        if what == "block":  # argument records of the products that share a launch
            s["jobs_qkv"], s["jobs_gate_up"] = rsr.make_jobs([s["q"], s["k"], s["v"]]), rsr.make_jobs([s["gate"], s["up"]])
    elif what == "qbit":
        q = case["bits"]
        A = torch.randint(-(1 << (q - 1)), 1 << (q - 1), (case["rows"], case["cols"]), generator=g, device="cuda", dtype=torch.int8)
        s["held"] = _Held(rsr.rsr_qbit_destroy)
        s["h"] = s["held"].add(rsr.rsr_qbit_preprocess(A.cpu().numpy(), case["k"], q))
        s["v"], s["out"] = _vectors(g, batch, case["rows"], dtype), _result(batch, case["cols"], dtype)
    elif what == "build":
        s["A"] = _matrix(g, case["kind"], case["rows"], case["cols"], case.get("zeros", 0.0))
        s["k"] = case["k"]
        s["v"], s["out"] = _vectors(g, batch, case["rows"], dtype), _result(batch, case["cols"], dtype)
    else:
        raise ValueError(what)
    torch.cuda.synchronize()
    return s


def run(s):
    what, batch, stream = s["what"], s["batch"], s["stream"]
    i8 = s["dtype"] == "i8"
    matvec = rsr.rsr_matvec_i8 if i8 else rsr.rsr_matvec
    if what == "product":
        matvec(s["h"], s["v"], s["out"], batch, stream)
        return s["out"]
    if what == "qbit":
        (rsr.rsr_qbit_matvec_i8 if i8 else rsr.rsr_qbit_matvec)(s["h"], s["v"], s["out"], batch, stream)
        return s["out"]
    if what == "stages":
        for name in STAGES:
            h, v, out = s[name]
            matvec(h, v, out, batch, stream)
        return [s[name][2] for name in STAGES]
    if what == "block":
        multi = rsr.rsr_matvec_multi_i8 if i8 else rsr.rsr_matvec_multi
        multi(s["jobs_qkv"], batch, stream)
        matvec(*s["o"], batch, stream)
        multi(s["jobs_gate_up"], batch, stream)
        matvec(*s["down"], batch, stream)
        return [s[name][2] for name in BLOCK]
    # build: index, product, and the index goes again (which waits for the product)
    A = s["A"]
    h = rsr.rsr_preprocess_device(A, A.shape[0], A.shape[1], s["k"])
    matvec(h, s["v"], s["out"], batch, stream)
    torch.cuda.current_stream().synchronize()
    rsr.rsr_destroy(h)
    return s["out"]


# ---- what a pass cannot do without -------------------------------------------------------------------------
def _product_work(parts, rows, cols, k, batch, dtype):
    """One reading of the permutations (16 bits per row, column block and part), activations in, results out; one addition
    per row, block and part, and the fold of 2^k segment sums (two additions each), for every vector."""
    blocks = -(-cols // k)
    return (parts * blocks * rows * 2 + batch * (rows * (1 if dtype == "i8" else 4) + cols * 4), batch * parts * blocks * (rows + 2 * 2**k))


def work(case):
    what, batch, dtype = case["what"], case["batch"], case["dtype"]
    if what in ("block", "stages"):
        each = [_product_work(2, rows, cols, case["k"], batch, dtype) for rows, cols in (BLOCK if what == "block" else STAGES).values()]
    elif what == "qbit":
        each = [_product_work(case["bits"], case["rows"], case["cols"], case["k"], batch, dtype)]
    else:
        each = [_product_work(1 if case["kind"] == "binary" else 2, case["rows"], case["cols"], case["k"], batch, dtype)]
        if what == "build":  # the matrix is read, the permutations are written
            blocks = -(-case["cols"] // case["k"])
            each.append((case["rows"] * case["cols"] + (1 if case["kind"] == "binary" else 2) * blocks * case["rows"] * 2, 0))
    return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}


def tolerance(case):
    """int8 products are exact.  Float products are sums of up to 32768 32-bit numbers: against the same products in 64 bits
    (_measure_tolerance) they were off by up to 1.5e-7 in the norm and 7.1e-7 of the larger of value and root mean square;
    about four times that is allowed, and a little more for weighted planes, whose partial products are larger than their sum."""
    if case["dtype"] == "i8":
        return "exact"
    return {"rel": 1e-6, "max": 5e-6} if case["what"] == "qbit" else {"rel": 6e-7, "max": 3e-6}


def _measure_tolerance():
    """Relative error of float products against the same products in 64 bits, over listed and drawn cases."""
    rng = random.Random(7)
    for case in listed() + [draw(rng) for _ in range(8)]:
        if case["what"] != "product" or case["dtype"] != "f32":
            continue
        g = _generator(11)
        A = _matrix(g, case["kind"], case["rows"], case["cols"], case.get("zeros", 0.0))
        h = _index(A, case["k"])
        v, out = _vectors(g, case["batch"], case["rows"], "f32"), _result(case["batch"], case["cols"], "f32")
        rsr.rsr_matvec(h, v, out, case["batch"], torch.cuda.current_stream().cuda_stream)
        step = max(1, (1 << 26) // case["rows"])
        exact = torch.cat([v.double() @ A[:, c:c + step].double() for c in range(0, case["cols"], step)], dim=1)
        torch.cuda.synchronize()
        rsr.rsr_destroy(h)
        off, rms = out.double() - exact, exact.square().mean().sqrt()
        worst = (off.abs() / torch.maximum(exact.abs(), rms)).max()
        print({k: case[k] for k in ("kind", "rows", "cols", "k", "batch")}, "rel %.3g" % float(off.norm() / exact.norm()), "max %.3g" % float(worst), flush=True)


if __name__ == "__main__":
    print("torch", torch.__version__)
    _measure_tolerance()
