"""The workloads whose speed is measured: what programs have this library do, through its public entry points.

Ranges: one biquaternion product in FP64 from a few rows to n = 8192, square and ragged, with every op; the
subalgebra entry points; the split-precision forms (CRT residues, INT8, BF16 and FP8 digits); batched plans of
uneven products in FP64 and in the CRT form; the diagonalization of a Hermitian matrix.  `listed` holds one case
of each use, `draw` gives more from the same ranges.  Inputs are drawn on the GPU from the seed: uniform [-1, 1]
and N(0, 1) entries, magnitudes spread over 1e-6..1e6, and Hermitian matrices with an exponentially decaying
spectrum (Fock- and density-like).  `exact` is the component-wise form, 64 real products in torch.
"""
import math
import random

import torch

import paper_2609_02081_amd as bq

UNIT_MASKS = {"biquaternion": 0xFF, "real_quaternion": 0x0F, "complex": 0x11, "real": 0x01}
REAL_GEMMS = {"biquaternion": 24, "real_quaternion": 8, "complex": 3, "real": 1}
COMPS = {a: [c for c in range(8) if m >> c & 1] for a, m in UNIT_MASKS.items()}
# CRT form: the moduli in the order they are used; digit forms: digit bits and headroom, most slices.
MODULI = (255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 211, 199, 197, 193, 191, 181, 179, 173, 167, 163)
DIGITS = {"split_bf16": (7, 0, 8), "split_fp8": (5, 1, 13), "split_int8": (7, 1, 9)}
# Quaternion units 1, i, j, k: e_u e_v = sign e_w.
UNITS = [[(1, 0), (1, 1), (1, 2), (1, 3)], [(1, 1), (-1, 0), (1, 3), (-1, 2)],
         [(1, 2), (-1, 3), (-1, 0), (1, 1)], [(1, 3), (1, 2), (-1, 1), (-1, 0)]]
OP_SIGNS = {"N": (1, 1, 1, 1), "T": (1, 1, -1, 1), "C": (1, -1, 1, -1), "H": (1, -1, -1, -1)}


def _gemm(name, m, k, n, opA="N", opB="N", dist="uniform", prec="fp64", entry="gemm", algebra="biquaternion"):
    case = dict(kind="gemm", entry=entry, algebra=algebra, m=m, k=k, n=n, opA=opA, opB=opB, dist=dist, prec=prec)
    return dict(case, name=name) if name else case


def _batch(name, count, lo, hi, prec, pick):
    case = dict(kind="batch", count=count, lo=lo, hi=hi, prec=prec, pick=pick)
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest ordinary call: one product inside a serving loop that may not allocate.
        _gemm("noalloc_64", 64, 64, 64, entry="noalloc"),
        # A single small product, uniform entries.
        _gemm("fp64_256", 256, 256, 256),
        # A ragged overlap A^dagger B of two rectangular blocks (stored transposed, odd row lengths).
        _gemm("fp64_ragged_HN", 1000, 777, 515, opA="H", dist="normal"),
        # An ordinary large product, N(0, 1) entries.
        _gemm("fp64_4096", 4096, 4096, 4096, dist="normal"),
        # A Fock matrix times a density matrix: the largest single product here.
        _gemm("fp64_8192_hermitian", 8192, 8192, 8192, dist="hermitian"),
        # Spinor rotations and other real-quaternion algebra through its own entry point.
        _gemm("real_quaternion_1024", 1024, 1024, 1024, entry="rq", algebra="real_quaternion"),
        # The CRT form: FP64-accurate products on the INT8 units, moderate and large.
        _gemm("crt_1024", 1024, 1024, 1024, prec="split_int8_crt"),
        _gemm("crt_4096", 4096, 4096, 4096, prec="split_int8_crt", dist="hermitian"),
        # The digit-slice form.
        _gemm("int8_digits_2048", 2048, 2048, 2048, prec="split_int8"),
        # Many independent products of uneven size in one graph launch.
        _batch("batch_fp64", 128, 64, 1536, "fp64", 5),
        _batch("batch_crt", 64, 64, 1536, "split_int8_crt", 6),
        # Eigenvalues and eigenvectors of a Hermitian matrix with every component present.
        dict(kind="heev", name="heev_256", n=256),
    ]


def _size(rng, lo, hi):
    """Log-uniform; three of ten are a multiple of 64, three more of 8, the rest as they fall."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    step = rng.choice((1, 1, 1, 1, 8, 8, 8, 64, 64, 64))
    return max(lo, min(hi, (v + step // 2) // step * step or v))


def draw(rng):
    use = rng.choice(("small", "single", "single", "single", "sub", "crt", "crt", "digits", "batch", "batch_crt", "heev"))
    dist = rng.choice(("uniform", "normal", "logspread"))
    opA, opB = rng.choice("NNNTCH"), rng.choice("NNNTCH")
    if use == "small":
        return _gemm(None, *(_size(rng, 8, 512) for _ in range(3)), opA, opB, dist, entry="noalloc")
    if use == "single":
        n = _size(rng, 16, 6000)
        if rng.random() < 0.4:
            return _gemm(None, n, n, n, opA, opB, dist)
        return _gemm(None, n, _size(rng, max(8, n // 4), min(6000, 4 * n)), _size(rng, max(8, n // 4), min(6000, 4 * n)),
                     opA, opB, dist)
    if use == "sub":
        entry = rng.choice(("rq", "cx", "re"))
        n = _size(rng, 32, 4096)
        algebra = {"rq": "real_quaternion", "cx": "complex", "re": "real"}[entry]
        return _gemm(None, n, _size(rng, max(8, n // 2), n), n, opA, opB, dist, entry=entry, algebra=algebra)
    if use == "crt":
        n = _size(rng, 64, 4096)
        return _gemm(None, n, _size(rng, max(16, n // 2), n), n, opA, opB, dist, prec="split_int8_crt")
    if use == "digits":
        n = _size(rng, 64, 3072)
        return _gemm(None, n, _size(rng, max(16, n // 2), n), n, opA, opB, dist,
                     prec=rng.choice(("split_int8", "split_bf16", "split_fp8")))
    if use == "heev":
        return dict(kind="heev", n=_size(rng, 32, 384))
    prec = "fp64" if use == "batch" else "split_int8_crt"
    hi = rng.choice((192, 384, 768, 1536))
    return _batch(None, rng.randint(8, 160 if hi < 1536 else 96), rng.choice((16, 64)), hi, prec, rng.randrange(1 << 20))


# ---- inputs -------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _entries(shape, dist, g):
    t = torch.empty(shape, dtype=torch.float64, device="cuda")
    if dist == "normal":
        return t.normal_(generator=g)
    if dist == "logspread":
        mag = torch.pow(10.0, t.uniform_(-6.0, 6.0, generator=g))
        return mag.mul_(torch.empty_like(mag).uniform_(-1.0, 1.0, generator=g).sign())
    return t.uniform_(-1.0, 1.0, generator=g)


def _hermitian(n, signed, g):
    """(8, n, n): the components of Z = U diag(lambda) U^H (2n x 2n, U four Householder reflectors, lambda from 1 down
    to 1e-8, with random signs for a Fock-like matrix), which satisfy A^dagger = A."""
    N = 2 * n
    lam = 10.0 ** torch.linspace(0.0, -8.0, N, dtype=torch.float64, device="cuda")
    if signed:
        lam = lam * torch.empty_like(lam).uniform_(-1.0, 1.0, generator=g).sign()
    Z = torch.diag(lam.to(torch.complex128))
    for _ in range(4):
        v = torch.complex(_entries((N,), "normal", g), _entries((N,), "normal", g))
        v /= torch.linalg.vector_norm(v)
        Z.addr_(v, v.conj() @ Z, alpha=-2.0)
        Z.addr_(Z @ v, v.conj(), alpha=-2.0)
    out = torch.empty((8, n, n), dtype=torch.float64, device="cuda")
    a, b, c, d = Z[:n, :n], Z[:n, n:], Z[n:, :n], Z[n:, n:]
    out[0], out[1] = 0.5 * (a.real + d.real), 0.5 * (a.imag - d.imag)
    out[2], out[3] = 0.5 * (b.real - c.real), 0.5 * (b.imag + c.imag)
    out[4], out[5] = 0.5 * (a.imag + d.imag), -0.5 * (a.real - d.real)
    out[6], out[7] = 0.5 * (b.imag - c.imag), -0.5 * (b.real + c.real)
    for u in range(8):  # the dagger's sign of each component, exactly
        s = 1.0 if u in (0, 5, 6, 7) else -1.0
        out[u] = 0.5 * (out[u] + s * out[u].T)
    return out


def _operands(case, seed):
    """A and B as stored (op T and H store the transpose): lists of 8 blocks, None where the algebra has none."""
    g = _gen(seed)
    m, k, n = case["m"], case["k"], case["n"]
    if case["dist"] == "hermitian":
        return list(_hermitian(n, True, g)), list(_hermitian(n, False, g))
    A = _entries((8, *((k, m) if case["opA"] in "TH" else (m, k))), case["dist"], g)
    B = _entries((8, *((n, k) if case["opB"] in "TH" else (k, n))), case["dist"], g)
    live = COMPS[case["algebra"]]
    return [A[c] if c in live else None for c in range(8)], [B[c] if c in live else None for c in range(8)]


def _sizes(case):
    r = random.Random(case["pick"])
    return [int(round(math.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]))))) for _ in range(case["count"])]


def _batch_inputs(case, seed):
    g = _gen(seed)
    return [(_entries((8, n, n), "uniform", g), _entries((8, n, n), "uniform", g)) for n in _sizes(case)]


# ---- the cases ----------------------------------------------------------------------------------------------------
def prepare(case, seed):
    state = {"case": case}
    if case["kind"] == "heev":
        state["A"] = _hermitian(case["n"], True, _gen(seed))
    elif case["kind"] == "batch":
        # One buffer for every result: a plan keeps the addresses of its operands.
        pairs = _batch_inputs(case, seed)
        out = torch.empty(sum(a.numel() for a, _ in pairs), dtype=torch.float64, device="cuda")
        triples, at = [], 0
        for a, b in pairs:
            triples.append((a, b, out[at:at + a.numel()].view(a.shape)))
            at += a.numel()
        plan = bq.GroupedPlan(triples, prec=case["prec"])
        plan.workspace()
        state.update(plan=plan, out=out)
    else:
        A, B = _operands(case, seed)
        live = COMPS[case["algebra"]]
        state["A"], state["B"] = (torch.stack(X) if len(live) == 8 else [X[c] for c in live] for X in (A, B))
        if case["entry"] != "gemm":
            state["C"] = torch.empty((len(live), case["m"], case["n"]), dtype=torch.float64, device="cuda")
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "heev":
        w, V, info = bq.heev(state["A"])
        return {"w": w, "V": V, "info": info}
    if case["kind"] == "batch":
        state["plan"].launch()
        return state["out"]
    A, B, ops = state["A"], state["B"], {"opA": case["opA"], "opB": case["opB"]}
    if case["entry"] == "gemm":
        return bq.bq_gemm(A, B, prec=case["prec"], **ops)
    if case["entry"] == "noalloc":
        return bq.bq_gemm_noalloc(A, B, state["C"], prec=case["prec"], **ops)
    C = state["C"]
    if case["entry"] == "rq":
        bq.rq_gemm(A, B, list(C), prec=case["prec"], **ops)
    elif case["entry"] == "cx":
        bq.cx_gemm(A, B, (C[0], C[1]), prec=case["prec"], **ops)
    else:
        bq.re_gemm(A[0], B[0], C[0], prec=case["prec"], **ops)
    return C


def _products(prec, k):
    """Low-precision GEMMs one real product of inner dimension k takes at the default slice or modulus count."""
    if prec == "fp64":
        return 1
    if prec == "split_int8_crt":
        have = 1
        for i, p in enumerate(MODULI):
            have *= p
            if have > 2 * k * 2 ** 106:
                return i + 1
        return len(MODULI)
    beta, head, most = DIGITS[prec]
    need = 48 + (max(0, (k - 1).bit_length()) + 1) // 2
    S = next((s for s in range(1, most + 1) if beta * s - head >= need), most)
    return S * (S + 1) // 2


def work(case):
    if case["kind"] == "heev":
        N = 2 * case["n"]  # reduction to tridiagonal form and back-transformation of the complex isomorph
        return {"bytes": 64.0 * case["n"] ** 2 + 16.0 * N * N + 8.0 * N, "flops": (16 / 3 + 8) * N ** 3}
    if case["kind"] == "batch":
        sizes = _sizes(case)
        return {"bytes": sum(24 * 8.0 * n * n for n in sizes),
                "flops": sum(24 * _products(case["prec"], n) * 2.0 * n ** 3 for n in sizes)}
    m, k, n, comps = case["m"], case["k"], case["n"], len(COMPS[case["algebra"]])
    return {"bytes": 8.0 * comps * (m * k + k * n + m * n),
            "flops": REAL_GEMMS[case["algebra"]] * _products(case["prec"], k) * 2.0 * m * n * k}


# ---- the same in plain torch --------------------------------------------------------------------------------------
def _op(X, op):
    out = []
    for c in range(8):
        if X[c] is None:
            out.append(None)
            continue
        s = OP_SIGNS[op][c % 4] * (-1 if c >= 4 and op in "CH" else 1)
        out.append(s * (X[c].T.contiguous() if op in "TH" else X[c]))
    return out


def _componentwise(A, B, m, n):
    """Sum over unit pairs of the products of (A_u + i A_u') and (B_v + i B_v'), one real product at a time."""
    C = torch.zeros((8, m, n), dtype=torch.float64, device="cuda")
    for u in range(4):
        for v in range(4):
            sign, w = UNITS[u][v]
            for ia in (0, 1):
                for ib in (0, 1):
                    a, b = A[u + 4 * ia], B[v + 4 * ib]
                    if a is not None and b is not None:
                        C[w + 4 * (ia ^ ib)].add_(torch.mm(a, b), alpha=-sign if ia and ib else sign)
    return C


def exact(case, seed):
    if case["kind"] == "heev":
        c = _hermitian(case["n"], True, _gen(seed)).cpu()
        Z = torch.cat([torch.cat([torch.complex(c[0] - c[5], c[1] + c[4]), torch.complex(c[2] - c[7], c[3] + c[6])], 1),
                       torch.cat([torch.complex(-c[2] - c[7], c[3] - c[6]), torch.complex(c[0] + c[5], c[4] - c[1])], 1)], 0)
        return {"w": torch.linalg.eigvalsh(Z), "V": None, "info": None}
    if case["kind"] == "batch":
        return torch.cat([_componentwise(list(a), list(b), a.shape[1], a.shape[1]).reshape(-1)
                          for a, b in _batch_inputs(case, seed)])
    A, B = _operands(case, seed)
    C = _componentwise(_op(A, case["opA"]), _op(B, case["opB"]), case["m"], case["n"])
    return C if case["entry"] in ("gemm", "noalloc") else C[COMPS[case["algebra"]]]
