"""The work that users have this library do, as cases that can be timed and compared.

Products ``C = A.B`` of multiple doubles through ``mdgemm_ex`` (1 to 16 limbs, every
pair set and width option that is used in earnest), the double-double Householder QR
(``mdgemm_qr_dd``) and the Taylor series of power-series systems (``mdgemm_taylor_dd``).
Sizes and values follow ``paper_2607_06881_amd/workloads.py``, the tests and ``bench.py``.

A case is a dict of plain values:

* ``op``: ``product``, ``qr`` or ``taylor``;
* products: ``limbs, m, n, k``, ``cutoff`` (``default`` or ``all``), ``mode`` (``pairs``:
  13-bit digits; ``auto``: the adaptive width; ``int8``; ``karatsuba``), ``range_bits``,
  ``base`` (``uniform`` or ``normal``), ``row_exp`` / ``elem_exp`` / ``inner_exp`` (power-of-two
  scales as in the workloads), ``workspace`` (the program keeps a workspace and passes it);
* qr: ``m, n``;  taylor: ``n, r, d``.
"""

import math

import torch

from paper_2607_06881_amd import mdgemm as md

DEV = "cuda"

_PRODUCT = {"op": "product", "cutoff": "default", "mode": "pairs", "range_bits": 0, "base": "uniform", "row_exp": 0,
            "elem_exp": 0, "inner_exp": 0, "workspace": False}


def _product(limbs, m, n, k, **more):
    return {**_PRODUCT, "limbs": limbs, "m": m, "n": n, "k": k, **more}


def listed():
    cases = {
        # the smallest product of the benchmark: one launch, latency counts
        "dd_64_all": _product(2, 64, 64, 64, cutoff="all"),
        # an ordinary call with odd sizes: a block of a larger computation
        "dd_ragged_small": _product(2, 333, 217, 501, base="normal"),
        # every digit pair kept, a workspace that the program keeps
        "dd_1024_all_workspace": _product(2, 1024, 1024, 1024, cutoff="all", row_exp=20, workspace=True),
        # the benchmark's headline product
        "dd_4096": _product(2, 4096, 4096, 4096, elem_exp=8),
        # quad double, as in the experiments with n = 2048
        "qd_2048": _product(4, 2048, 2048, 1024, base="normal"),
        # the largest output: a short inner dimension under a wide C
        "td_8192": _product(3, 8192, 8192, 512, base="normal", row_exp=30),
        # hexa double: the most limbs, a thin A
        "hd_thin": _product(16, 128, 8192, 64, base="normal"),
        # lines of a wide range, balanced with more digits
        "dd_2048_range": _product(2, 2048, 2048, 2048, base="normal", inner_exp=60, range_bits=60),
        # the int8 level products that a caller can choose, with odd sizes
        "dd_3001_int8": _product(2, 3001, 2999, 4097, mode="int8"),
        # the adaptive width, with odd sizes and a workspace that the program keeps
        "dd_1777_auto_workspace": _product(2, 1777, 2049, 1531, mode="auto", base="normal", workspace=True),
        # the factorization of a double-double matrix, whose updates are products
        "qr_2048": {"op": "qr", "m": 2048, "n": 2048},
        # the series solution of a linear system: one QR, then products per degree
        "taylor_1024": {"op": "taylor", "n": 1024, "r": 64, "d": 8},
    }
    return [{"name": name, **case} for name, case in cases.items()]


# digit pairs of the default 13-bit digits, for bounding a drawn case's cost
def _digits(limbs):
    return 4 * limbs if limbs <= 4 else math.ceil((53 * limbs - 4) / 13) + 1


def _log(rng, lo, hi):
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(max(x | 1 if rng.random() < 0.5 else x, lo), hi)


def draw(rng):
    kind = rng.random()
    if kind < 0.08:
        n = _log(rng, 32, 2048)
        return {"op": "qr", "m": min(2 * n, n + _log(rng, 1, 512)) if rng.random() < 0.5 else n, "n": n}
    if kind < 0.16:
        return {"op": "taylor", "n": _log(rng, 16, 1024), "r": _log(rng, 1, 64), "d": rng.randint(0, 8)}
    limbs = rng.choice([1, 2, 2, 2, 2, 3, 3, 4, 4, 8, 16])
    most = 36 * 4096 ** 3
    while True:
        m, n, k = _log(rng, 16, 8192), _log(rng, 16, 8192), _log(rng, 16, 4096)
        s = _digits(limbs)
        cutoff = "all" if rng.random() < 0.2 else "default"
        pairs = s * s if cutoff == "all" else s * (s + 1) // 2
        if pairs * m * n * k <= most and limbs * m * n <= 3 * 8192 ** 2:
            break
    mode = rng.choice(["pairs", "pairs", "pairs", "auto", "int8" if limbs <= 8 else "pairs", "karatsuba"])
    case = _product(limbs, m, n, k, cutoff=cutoff, mode=mode, base=rng.choice(["uniform", "normal"]),
                    row_exp=rng.choice([0, 0, 20, 30]), elem_exp=rng.choice([0, 0, 8]),
                    workspace=rng.random() < 0.35)
    if limbs <= 3 and cutoff == "default" and rng.random() < 0.15:
        case.update(inner_exp=60, range_bits=60, elem_exp=0, m=min(m, 2048), n=min(n, 2048), k=min(k, 2048))
    return case


def _two_sum(a, b):
    s = a + b
    bb = s - a
    return s, (a - (s - bb)) + (b - bb)


def _operand(g, limbs, rows, cols, base, row_exp=0, col_exp=0, elem_exp=0):
    """A normalized multiple-double matrix [limbs, rows, cols] (see workloads.make_operand)."""
    x = torch.empty((limbs, rows, cols), dtype=torch.float64, device=DEV)
    if base == "normal":
        x[0].normal_(generator=g)
    else:
        x[0].uniform_(-1.0, 1.0, generator=g)
    for i in range(1, limbs):
        x[i].uniform_(-1.0, 1.0, generator=g).mul_(x[i - 1]).mul_(2.0 ** -53)
    for _ in range(2 if limbs > 2 else 1):  # exact sweeps that make the limbs nonoverlapping
        for i in list(range(limbs - 1)) + list(range(limbs - 2, -1, -1)):
            s, e = _two_sum(x[i], x[i + 1])
            x[i].copy_(s)
            x[i + 1].copy_(e)
    for exp, shape in ((row_exp, (rows, 1)), (col_exp, (1, cols)), (elem_exp, (rows, cols))):
        if exp:
            e = torch.randint(-exp, exp + 1, shape, device=DEV, generator=g)
            x.mul_(torch.pow(2.0, e.to(torch.float64)))
    return x


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if case["op"] == "qr":
        return (_operand(g, 2, case["m"], case["n"], "uniform", elem_exp=8),)
    if case["op"] == "taylor":
        n, r, d = case["n"], case["r"], case["d"]
        a = torch.stack([_operand(g, 2, n, n, "normal") for _ in range(d + 1)])
        a.mul_(2.0 ** -round(math.log2(math.sqrt(n))))
        # a well-conditioned leading coefficient: the diagonal moved by 2 (exactly)
        diag = torch.diagonal(a[0, 0]), torch.diagonal(a[0, 1])
        s, e = _two_sum(torch.full_like(diag[0], 2.0), diag[0])
        s, e = _two_sum(s, e + diag[1])
        diag[0].copy_(s)
        diag[1].copy_(e)
        return a, torch.stack([_operand(g, 2, n, r, "normal") for _ in range(d + 1)])
    L, m, n, k = case["limbs"], case["m"], case["n"], case["k"]
    a = _operand(g, L, m, k, case["base"], row_exp=case["row_exp"], elem_exp=case["elem_exp"])
    b = _operand(g, L, k, n, case["base"], col_exp=case["row_exp"], elem_exp=case["elem_exp"])
    if case["inner_exp"]:
        e = torch.randint(0, case["inner_exp"] + 1, (k,), device=DEV, generator=g).to(torch.float64)
        a.mul_(torch.pow(2.0, -e)[None, None, :])
        b.mul_(torch.pow(2.0, e - case["inner_exp"])[None, :, None])
    return a, b


def _options(case):
    opts = {}
    if case["cutoff"] == "all":
        opts["cutoff"] = md.MDGEMM_CUTOFF_ALL
    if case["range_bits"]:
        opts["range_bits"] = case["range_bits"]
    if case["mode"] == "auto":
        opts["slice_bits"] = md.MDGEMM_SLICE_BITS_AUTO
    elif case["mode"] == "int8":
        opts["flags"] = md.MDGEMM_INT8
    elif case["mode"] == "karatsuba":
        opts["flags"] = md.MDGEMM_KARATSUBA
    return opts


def prepare(case, seed):
    state = {"op": case["op"], "in": _inputs(case, seed)}
    if case["op"] == "qr":
        m, n = case["m"], case["n"]
        state["work"] = torch.empty_like(state["in"][0])
        state["ws"] = torch.empty(int(md.lib().mdgemm_qr_dd_workspace_bytes(m, n, 64)), dtype=torch.uint8, device=DEV)
    elif case["op"] == "taylor":
        need = int(md.lib().mdgemm_taylor_dd_workspace_bytes(case["n"], case["r"], case["d"]))
        state["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        state["x"] = torch.empty_like(state["in"][1])
    else:
        L, m, n, k = case["limbs"], case["m"], case["n"], case["k"]
        opts = _options(case)
        if case["workspace"]:
            need = md.mdgemm_workspace_bytes(m, n, k, L, **opts)
            opts["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        state["opts"] = opts
        state["c"] = torch.empty((L, m, n), dtype=torch.float64, device=DEV)
    return state


def run(state):
    if state["op"] == "qr":
        state["work"].copy_(state["in"][0])  # the factorization works in place
        a, tau = md.mdgemm_qr_dd(state["work"], workspace=state["ws"])
        return {"high": a[0], "low": a[1], "tau": tau[0], "tau_low": tau[1]}
    if state["op"] == "taylor":
        a, b = state["in"]
        x = md.mdgemm_taylor_dd(a, b, X=state["x"], workspace=state["ws"])
        return {"high": x[:, 0], "low": x[:, 1]}
    a, b = state["in"]
    c = md.mdgemm_ex(a, b, state["c"], **state["opts"])
    return {"high": c[0], "low": c[1:]} if c.shape[0] > 1 else {"high": c[0]}


def work(case):
    """Operands read once and the result written once; a multiple-double product
    as its limb pairs down to the last limb of the result (L (L + 1) / 2 of them, all L^2 with
    every digit pair kept)."""
    if case["op"] == "qr":
        m, n = case["m"], case["n"]
        return {"bytes": 2 * 8.0 * 2 * m * n, "flops": 3 * (2.0 * m * n * n - 2.0 * n ** 3 / 3)}
    if case["op"] == "taylor":
        n, r, d = case["n"], case["r"], case["d"]
        flops = 2.0 * n ** 3 * 2 / 3 + (d + 1) * 2.0 * n * n * r + d * (d + 1) / 2 * 2.0 * n * n * r
        return {"bytes": 16.0 * (d + 1) * n * (n + 2 * r), "flops": 3 * flops}
    L, m, n, k = case["limbs"], case["m"], case["n"], case["k"]
    pairs = L * L if case["cutoff"] == "all" else L * (L + 1) // 2
    return {"bytes": 8.0 * L * (m * k + k * n + m * n), "flops": 2.0 * pairs * m * n * k}


def tolerance(case):
    # a product's limbs are the greedy rounding of an exact integer: no other answer is right
    if case["op"] == "product":
        return "exact"
    # Double-double chains.  Four times and more of what other panel widths (QR: low limbs up to
    # 9e-14 of their norm, 2.7e-12 of the largest entry) and a permuted system (Taylor: 7e-13,
    # 4.7e-12) change; the condition of a random square matrix varies by some factors from draw to draw.
    return {"rel": 2e-12, "max": 4e-11} if case["op"] == "qr" else {"rel": 3e-12, "max": 2e-11}


def exact(case, seed):
    """The leading limbs in float64 from plain torch; the lower limbs have no value in 64 bits."""
    if case["op"] == "product":
        if case["m"] * case["n"] * case["k"] > 4096 ** 3:
            return None
        a, b = _inputs(case, seed)
        c = a[0].cpu() @ b[0].cpu() if a.shape[1] * b.shape[2] * a.shape[2] < 2 ** 31 else a[0] @ b[0]
        return {"high": c, "low": None} if case["limbs"] > 1 else {"high": c}
    if case["op"] == "taylor":
        a, b = (x[:, 0].cpu() for x in _inputs(case, seed))
        inv, x = torch.linalg.inv(a[0]), []
        for i in range(case["d"] + 1):
            rhs = b[i].clone()
            for j in range(1, i + 1):
                rhs -= a[j] @ x[i - j]
            x.append(inv @ rhs)
        return {"high": torch.stack(x), "low": None}
    return None  # the vectors and R of another factorization differ in rounding by the matrix's condition
