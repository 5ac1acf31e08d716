"""The work a user of this library has it do, as cases that can be timed.

A case names an entry point, a shape and the options of one emulated FP64
product (or of one batch of products).  `listed` holds the cases by name,
`draw` gives further ones from the same ranges, `prepare` makes what a program
has in hand before the call, `run` is one call, `work` is what the call cannot
do without and `exact` is the same product in plain float64.
"""
import math
import random

import torch

import paper_2603_10634_amd as oz

# digit products per modulus: three FP8 products (square or Karatsuba split),
# or one INT8 product
_PRODUCTS = {"hybrid": 3, "int8": 1}

_DEFAULTS = {"entry": "blas", "transA": "N", "transB": "N", "N": 12, "moduli": "hybrid",
             "mode": "accurate", "phi": 0.5, "alpha": 1.0, "beta": 0.0, "pad": 0, "graph": False}


def _case(**kw):
    return {**_DEFAULTS, **kw}


def listed():
    return [
        # the smallest calls: a loop over small products, replayed from a
        # graph because launches are all it costs
        _case(name="graph_100x60x75", m=100, n=60, k=75, graph=True),
        # the 256^3 row-major product through the tensor wrapper
        _case(name="row_major_256", entry="rows", m=256, n=256, k=256),
        # trailing update of a blocked factorization: C <- C - A B inside
        # larger arrays, short k
        _case(name="update_3000x2000x256", m=3000, n=2000, k=256, alpha=-1.0, beta=1.0, pad=72,
              phi=1.0),
        # an odd product under the no-allocation entry point, wider inputs
        _case(name="noalloc_1111x777x1999", entry="noalloc", m=1111, n=777, k=1999, transA="T",
              N=14, phi=2.0),
        # mid-size square product, fast mode at its own moduli count
        _case(name="fast_2048", m=2048, n=2048, k=2048, mode="fast", N=13),
        # the square workload at its smaller size
        _case(name="square_4096", m=4096, n=4096, k=4096),
        # the square workload at the headline size
        _case(name="square_8192", m=8192, n=8192, k=8192),
        # long contraction with a small result (normal equations, overlaps)
        _case(name="k_long_1024x1024x65536", m=1024, n=1024, k=65536, transA="T", phi=1.0),
        # large result from a short contraction (rank-k update)
        _case(name="k_short_16384x16384x1024", m=16384, n=16384, k=1024, phi=1.0),
        # odd sizes, wide dynamic range and the moduli count it needs
        _case(name="wide_3001x2777x3333", m=3001, n=2777, k=3333, transB="T", N=17, phi=4.0),
        # the INT8 moduli list
        _case(name="int8_4096", m=4096, n=4096, k=4096, moduli="int8", N=14),
        # many uneven products in one call
        _case(name="batched_48", entry="batched", count=48, lo=64, hi=2048, shapes=4, phi=1.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    trans = {"transA": rng.choice("NT"), "transB": rng.choice("NT")}
    scal = rng.choice([{}, {}, {"alpha": -1.0, "beta": 1.0}, {"alpha": 0.5, "beta": -0.25}])
    acc = rng.choice([{"N": 12}, {"N": 12, "phi": 1.0}, {"N": 13, "mode": "fast"},
                      {"N": 14, "phi": 2.0}, {"N": 17, "phi": 4.0}, {"N": 14, "moduli": "int8"}])
    kind = rng.choice(["small", "mid", "mid", "large", "k_long", "k_short", "batched"])
    if kind == "small":
        return _case(m=_log(rng, 33, 600), n=_log(rng, 33, 600), k=_log(rng, 33, 600),
                     graph=rng.random() < 0.5, pad=rng.choice([0, 5]), **trans, **scal, **acc)
    if kind == "mid":
        m, n, k = (_log(rng, 300, 3500) for _ in range(3))
        entry = "noalloc" if max(m, n, k) < 1100 else rng.choice(["blas", "rows"])
        if entry == "rows":
            return _case(entry="rows", m=m, n=n, k=k, **acc)
        return _case(entry=entry, m=m, n=n, k=k, pad=rng.choice([0, 7]), **trans, **scal, **acc)
    if kind == "large":
        return _case(m=_log(rng, 3000, 7000), n=_log(rng, 3000, 7000), k=_log(rng, 2000, 7000),
                     **trans, **acc)
    if kind == "k_long":
        return _case(m=_log(rng, 128, 1500), n=_log(rng, 128, 1500), k=_log(rng, 8192, 65536),
                     **trans, **acc)
    if kind == "k_short":
        return _case(m=_log(rng, 2000, 14000), n=_log(rng, 2000, 14000), k=_log(rng, 100, 1024),
                     **trans, **scal, **acc)
    return _case(entry="batched", count=rng.randint(6, 48), lo=64, hi=rng.choice([512, 1024, 2048]),
                 shapes=rng.randrange(1 << 20), phi=1.0)


def _batch_shapes(case):
    """(m, n, k) of every product, each log-uniform in [lo, hi]."""
    rng = random.Random(case["shapes"])
    return [tuple(_log(rng, case["lo"], case["hi"]) for _ in range(3))
            for _ in range(case["count"])]


def _draws(rows, cols, phi, gen):
    """rows x cols of (U - 0.5) exp(phi N(0, 1)) on the GPU."""
    u = torch.rand((rows, cols), dtype=torch.float64, device="cuda", generator=gen).sub_(0.5)
    g = torch.randn((rows, cols), dtype=torch.float64, device="cuda", generator=gen)
    return u.mul_(g.mul_(phi).exp_())


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    phi = case["phi"]
    if case["entry"] == "batched":
        shapes = _batch_shapes(case)
        return {"case": case,
                "A": [_draws(m, k, phi, gen) for m, n, k in shapes],
                "B": [_draws(k, n, phi, gen) for m, n, k in shapes]}
    m, n, k, pad = case["m"], case["n"], case["k"], case["pad"]
    if case["entry"] == "rows":
        return {"case": case, "A": _draws(m, k, phi, gen), "B": _draws(k, n, phi, gen)}
    # column-major arrays: a row of the tensor is a column of the matrix
    colsA, lda = (k, m + pad) if case["transA"] == "N" else (m, k + pad)
    colsB, ldb = (n, k + pad) if case["transB"] == "N" else (k, n + pad)
    A = _draws(colsA, lda, phi, gen)
    B = _draws(colsB, ldb, phi, gen)
    C = (_draws(n, m + pad, phi, gen) if case["beta"] else
         torch.zeros((n, m + pad), dtype=torch.float64, device="cuda"))
    return {"case": case, "A": A, "B": B, "C": C, "ld": (lda, ldb, m + pad)}


def run(state):
    case = state["case"]
    oz.ozaki2_set_moduli_list(case["moduli"])
    oz.ozaki2_set_graph(case["graph"])
    if case["entry"] == "batched":
        return oz.dgemm_batched(state["A"], state["B"], case["N"], mode=case["mode"])
    if case["entry"] == "rows":
        return oz.dgemm(state["A"], state["B"], case["N"], mode=case["mode"])
    oz.ozaki2_set_mode(case["mode"])
    oz.ozaki2_set_stream(torch.cuda.current_stream())
    call = oz.ozaki2_dgemm_noalloc if case["entry"] == "noalloc" else oz.ozaki2_dgemm
    lda, ldb, ldc = state["ld"]
    st = call(case["transA"], case["transB"], case["m"], case["n"], case["k"], case["alpha"],
              state["A"], lda, state["B"], ldb, case["beta"], state["C"], ldc, case["N"])
    oz.ozaki2_set_mode("accurate")
    if st != 0:
        raise oz.Ozaki2Error("ozaki2_dgemm", st)
    return state["C"][:, :case["m"]]


def work(case):
    """Operands read once (C too with beta), the result written once, and the
    digit products of every modulus."""
    shapes = (_batch_shapes(case) if case["entry"] == "batched" else
              [(case["m"], case["n"], case["k"])])
    c = 2 if case["beta"] else 1
    products = _PRODUCTS[case["moduli"]] * case["N"]
    return {"bytes": sum(8 * (m * k + k * n + c * m * n) for m, n, k in shapes),
            "flops": sum(2 * products * m * n * k for m, n, k in shapes)}


def exact(case, seed):
    s = prepare(case, seed)
    if case["entry"] == "batched":
        return [a @ b for a, b in zip(s["A"], s["B"])]
    if case["entry"] == "rows":
        return s["A"] @ s["B"]
    m, n, k = case["m"], case["n"], case["k"]
    # opA (m x k) and opB (k x n) as views of the column-major arrays
    opA = s["A"][:, :m].T if case["transA"] == "N" else s["A"][:, :k]
    opB = s["B"][:, :k].T if case["transB"] == "N" else s["B"][:, :n]
    C = case["alpha"] * (opB.T @ opA.T)
    return C + case["beta"] * s["C"][:, :m] if case["beta"] else C
