"""CRT-based split form (Ozaki scheme II) on the GPU, through the C-ABI.

Each real product of this form is the correctly rounded value of the product
of the scaled integers (the residues are reduced exactly and P is rounded to
FP64 once), so:

* one real product (masks with only the real unit component): bit-exact with
  oracle/ozaki2.product, which forms P with Python integers;
* integer inputs: bit-exact with the FP64 oracle (nothing rounds);
* random biquaternions: equal to the CPU split model (the bilinear scheme
  with ozaki2.product as the real GEMM) to 1e-14 relative, the two differing
  only in the FP64 order of the pre- and post-combination sums;
* default moduli: relative Frobenius error <= 1e-12 against the FP64 oracle.
"""
import numpy as np
import pytest

import oracle
from bilinear_model import Counter, bilinear
from oracle import ozaki2
from paper_2609_02081_amd import inputs

pytestmark = pytest.mark.gpu
TOL = 1e-12
PREC = "split_int8_crt"
OP_FN = {"N": lambda M: M, "T": oracle.transpose, "C": oracle.conj, "H": oracle.herm}


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_02081_amd as bq

    bq.lib()
    return bq


def run(bq, A, B, N=0, **kw):
    import torch

    C = bq.bq_gemm(torch.from_numpy(A).to("cuda"), torch.from_numpy(B).to("cuda"), prec=PREC, slices=N, **kw)
    torch.cuda.synchronize()
    return C.cpu().numpy()


@pytest.mark.parametrize("tile", ["128", "256"])
@pytest.mark.parametrize("dist", ["uniform", "logspread", "normal"])
@pytest.mark.parametrize("N", [0, 9, 20])
def test_real_product_bit_exact(bq, dist, N, tile, monkeypatch):
    """m, k, n = 300, 200, 70 with either residue-GEMM block: several row
    tiles with a ragged last one, ragged columns, k two 128-steps with a
    ragged tail: every element equal to the oracle's."""
    monkeypatch.setenv("BQ_CRT_TILE", tile)
    R = inputs.MASKS["real"]
    A, B = inputs.pair(300, 200, 70, dist, seed=60, mask_a=R, mask_b=R)
    print(f"crt real product {dist} N={N} tile {tile}", flush=True)
    got = run(bq, A, B, N, mask_a=R, mask_b=R)
    assert np.array_equal(got[0], ozaki2.product(A[0], B[0], N))
    assert not np.any(got[1:])


@pytest.mark.parametrize("N", [2, 4, 6])
def test_few_moduli_bit_exact(bq, N):
    """Few moduli carry few bits: the rounding of the inputs to b-bit
    integers dominates and must match the oracle exactly."""
    R = inputs.MASKS["real"]
    A, B = inputs.pair(40, 64, 33, "uniform", seed=61, mask_a=R, mask_b=R)
    assert ozaki2.bits_for(N, 64) >= 1
    got = run(bq, A, B, N, mask_a=R, mask_b=R)
    assert np.array_equal(got[0], ozaki2.product(A[0], B[0], N))


def test_integer_bit_exact(bq):
    A, B = inputs.pair(96, 80, 72, "int", seed=62, bound=64)
    print("crt integer", flush=True)
    assert np.array_equal(run(bq, A, B), oracle.gemm(A, B))


@pytest.mark.parametrize("tile", ["128", "256"])
@pytest.mark.parametrize("N", [0, 12])
def test_matches_cpu_split_model(bq, N, tile, monkeypatch):
    monkeypatch.setenv("BQ_CRT_TILE", tile)
    A, B = inputs.pair(70, 60, 50, "logspread", seed=63)
    print(f"crt N={N} vs model", flush=True)
    ref = bilinear(A, B, Counter(lambda x, y: ozaki2.product(x, y, N)))
    assert oracle.rel_frobenius(run(bq, A, B, N), ref) <= 1e-14


@pytest.mark.parametrize("dist", ["uniform", "logspread"])
def test_default_moduli_accuracy(bq, dist):
    A, B = inputs.pair(256, 256, 256, dist, seed=4)
    err = oracle.rel_frobenius(run(bq, A, B), oracle.gemm(A, B))
    print(f"crt default moduli, {dist}: rel err {err:.3e}", flush=True)
    assert err <= TOL


@pytest.mark.parametrize("opA,opB", [("T", "H"), ("H", "N"), ("N", "T"), ("C", "C")])
def test_ops_integer_bit_exact(bq, opA, opB):
    rng = np.random.default_rng(64)
    m, k, n = 96, 80, 72
    A = inputs.blocks(rng, *((k, m) if opA in "TH" else (m, k)), "int", bound=64)
    B = inputs.blocks(rng, *((n, k) if opB in "TH" else (k, n)), "int", bound=64)
    print(f"crt ops {opA}{opB} integer", flush=True)
    got = run(bq, A, B, opA=opA, opB=opB)
    assert np.array_equal(got, oracle.gemm(OP_FN[opA](A), OP_FN[opB](B)))


def test_ops_match_cpu_split_model(bq):
    rng = np.random.default_rng(65)
    m, k, n = 70, 60, 50
    A = inputs.blocks(rng, k, m, "logspread")   # stored for op H
    B = inputs.blocks(rng, n, k, "logspread")   # stored for op T
    ref = bilinear(oracle.herm(A), oracle.transpose(B), Counter(lambda x, y: ozaki2.product(x, y, 0)))
    assert oracle.rel_frobenius(run(bq, A, B, opA="H", opB="T"), ref) <= 1e-14


@pytest.mark.parametrize("mask", [0x0F, 0x11, 0x5A, 0x0E])
def test_masks(bq, mask):
    A, B = inputs.pair(90, 70, 60, "normal", seed=66, mask_a=mask, mask_b=mask)
    got = run(bq, A, B, mask_a=mask, mask_b=mask)
    assert oracle.rel_frobenius(got, oracle.gemm(A, B)) <= TOL


def test_zero_rows_columns_and_degenerate_shapes(bq):
    """A zero row of A and a zero column of B (no exponent) give zero rows
    and columns of the product; k = 1; k = 0 writes zeros."""
    R = inputs.MASKS["real"]
    A, B = inputs.pair(33, 65, 17, "uniform", seed=67, mask_a=R, mask_b=R)
    A[0, 5, :] = 0.0
    B[0, :, 3] = 0.0
    got = run(bq, A, B, mask_a=R, mask_b=R)
    assert np.array_equal(got[0], ozaki2.product(A[0], B[0]))
    assert not np.any(got[0][5, :]) and not np.any(got[0][:, 3])
    A1, B1 = inputs.pair(7, 1, 9, "uniform", seed=68)
    assert oracle.rel_frobenius(run(bq, A1, B1), oracle.gemm(A1, B1)) <= 1e-14
    A0, B0 = np.zeros((8, 5, 0)), np.zeros((8, 0, 6))
    assert not np.any(run(bq, A0, B0))


@pytest.mark.parametrize("tile", ["128", "256"])
def test_int32_sums_at_max_k(bq, tile, monkeypatch):
    """k = 133120, the largest k the form takes: every row of A and column of
    B equals 251/256, whose scaled integer 251 2^45 is 127 modulo 255, so the
    INT8 GEMM of that modulus sums k 127^2 = 2147092480 (just under 2^31).
    The product k (251/256)^2 is exact in FP64."""
    import torch

    monkeypatch.setenv("BQ_CRT_TILE", tile)
    k = 133120
    x = 251.0 / 256.0
    A = torch.zeros((8, 4, k), dtype=torch.float64, device="cuda")
    B = torch.zeros((8, k, 4), dtype=torch.float64, device="cuda")
    A[0].fill_(x)
    B[0].fill_(x)
    R = inputs.MASKS["real"]
    print("crt k=133120 worst-case int32 sums", flush=True)
    C = bq.bq_gemm(A, B, mask_a=R, mask_b=R, prec=PREC)
    torch.cuda.synchronize()
    assert torch.all(C[0] == k * x * x).item()
    assert ozaki2.residues(np.array([251 << 45]), 255)[0] == 127


def _sample(n, r, seed):
    rng = np.random.default_rng(seed)
    idx = np.sort(rng.choice(n - 1, size=r - 1, replace=False))
    return np.append(idx, n - 1)


@pytest.mark.parametrize("dist", ["uniform", "logspread"])
def test_n8192_sampled(bq, dist):
    """Default block choice (256 x 256 at this size)."""
    import torch

    n, r = 8192, 48
    rng = np.random.default_rng(4)
    print(f"crt n=8192 {dist}: inputs", flush=True)
    if dist == "uniform":
        A = inputs.device_uniform(n, n, 41, "cuda")
        B = inputs.device_uniform(n, n, 42, "cuda")
    else:
        A = torch.from_numpy(inputs.blocks(rng, n, n, "logspread")).to("cuda")
        B = torch.from_numpy(inputs.blocks(rng, n, n, "logspread")).to("cuda")
    C = bq.bq_gemm(A, B, prec=PREC)
    torch.cuda.synchronize()
    rows, cols = _sample(n, r, 51), _sample(n, r, 52)
    ri, ci = torch.as_tensor(rows, device="cuda"), torch.as_tensor(cols, device="cuda")
    As, Bs = A[:, ri, :].cpu().numpy(), B[:, :, ci].cpu().numpy()
    Cs = C[:, ri][:, :, ci].cpu().numpy()
    err = oracle.rel_frobenius(Cs, oracle.gemm(As, Bs))
    print(f"crt n=8192 {dist}: sampled rel err {err:.3e}", flush=True)
    assert err <= TOL


def test_real_product_n8192_sampled_bit_exact(bq):
    """At n = 8192 with the default 15 moduli (k = 8192), sampled elements of
    one real product equal the oracle's exactly."""
    import torch

    n, r = 8192, 6
    R = inputs.MASKS["real"]
    A = inputs.device_uniform(n, n, 43, "cuda")
    B = inputs.device_uniform(n, n, 44, "cuda")
    C = bq.bq_gemm(A, B, mask_a=R, mask_b=R, prec=PREC)
    torch.cuda.synchronize()
    rows, cols = _sample(n, r, 53), _sample(n, r, 54)
    ri, ci = torch.as_tensor(rows, device="cuda"), torch.as_tensor(cols, device="cuda")
    X = A[0][ri, :].cpu().numpy()
    Y = B[0][:, ci].cpu().numpy()
    # the exponents are per whole row of A and column of B: the sampled rows
    # and columns carry theirs, so the sampled product is the full product's
    want = ozaki2.product(X, Y, ozaki2.default_moduli(n))
    assert np.array_equal(C[0][ri][:, ci].cpu().numpy(), want)


@pytest.mark.parametrize("prec", ["split_int8_crt", "split_int8", "split_bf16", "split_fp8"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_propagation(bq, prec, bad):
    """A NaN or infinity in row 11 of A (component 7) and column 5 of B
    (component 2) makes row 11 and column 5 of every output component NaN,
    as in the FP64 path (there an infinity can also give +-inf); the rest
    stays finite and matches the oracle."""
    import torch

    A, B = inputs.pair(40, 40, 40, "uniform", seed=10)
    A[6, 11, 3] = bad
    B[1, 7, 5] = bad
    C = bq.bq_gemm(torch.from_numpy(A).to("cuda"), torch.from_numpy(B).to("cuda"), prec=prec)
    torch.cuda.synchronize()
    C = C.cpu().numpy()
    assert np.all(np.isnan(C[:, 11, :])) and np.all(np.isnan(C[:, :, 5]))
    rest = np.delete(np.delete(C, 11, axis=1), 5, axis=2)
    assert np.all(np.isfinite(rest))
    A2, B2 = A.copy(), B.copy()
    A2[6, 11, 3] = 0.0
    B2[1, 7, 5] = 0.0
    ref = np.delete(np.delete(oracle.gemm(A2, B2), 11, axis=1), 5, axis=2)
    assert oracle.rel_frobenius(rest, ref) <= TOL


def test_n24576_hermitian_sampled(bq):
    """n = 24576 in the CRT form (one FP64 block is 4.8 GB > 2^32 bytes, one
    residue plane 604 MB, the residue GEMM offsets run past 2^32): Fock-like
    A times density-like B against the oracle on sampled rows and columns
    that include the last ones."""
    import torch

    n = 24576
    print(f"crt n={n}: building Hermitian inputs on the device", flush=True)
    A, B = inputs.hermitian_pair(n, 3, "cuda")
    torch.cuda.empty_cache()  # the builder's temporaries, before the workspace
    C = bq.bq_gemm(A, B, prec=PREC)
    torch.cuda.synchronize()
    print(f"crt n={n}: product done", flush=True)
    r = 48
    rows, cols = _sample(n, r, 33), _sample(n, r, 34)
    ri, ci = torch.as_tensor(rows, device="cuda"), torch.as_tensor(cols, device="cuda")
    As = A[:, ri, :].cpu().numpy()
    Bs = B[:, :, ci].cpu().numpy()
    Cs = C[:, ri][:, :, ci].cpu().numpy()
    del A, B, C
    torch.cuda.empty_cache()
    err = oracle.rel_frobenius(Cs, oracle.gemm(As, Bs))
    print(f"crt n={n}: sampled rel err {err:.3e}", flush=True)
    assert err <= TOL


@pytest.mark.parametrize("m,k,n,tile", [(130, 70, 900, "128"), (385, 100, 129, "128"), (1290, 40, 520, "256"),
                                        (2600, 2400, 1500, "128")])
def test_residue_gemm_tile_order(bq, monkeypatch, m, k, n, tile):
    """Tile counts that are no multiple of 8, small planes (an XCD takes runs
    over moduli and tiles) and planes above 9 MiB (runs within each modulus):
    every tile of every modulus is formed once, so an integer product is the
    oracle's, checked on sampled rows and columns for the largest."""
    monkeypatch.setenv("BQ_CRT_TILE", tile)
    print(f"residue GEMM tile order {m}x{k}x{n} tile {tile}", flush=True)
    A, B = inputs.pair(m, k, n, "int", seed=91, bound=512)
    got = run(bq, A, B)
    rows = np.arange(0, m, max(1, m // 150))
    assert np.array_equal(got[:, rows], oracle.gemm(A[:, rows], B))


@pytest.mark.parametrize("m,k,n", [(1, 1, 1), (128, 128, 128), (257, 129, 129), (300, 200, 70), (900, 300, 1000)])
@pytest.mark.parametrize("tile", ["128", "256x128"])
def test_tiles_in_a_row(bq, monkeypatch, m, k, n, tile):
    """Tiles of 128 x 128 and 256 x 128: one tile a block, two k-steps (the
    loads run to the next tile from the first step on), ragged rows and
    columns, and more tiles than the 512 blocks of a launch, some with a
    second tile and some without.  An integer product is the oracle's."""
    monkeypatch.setenv("BQ_CRT_TILE", tile)
    print(f"residue tiles in a row {m}x{k}x{n} tile {tile}", flush=True)
    A, B = inputs.pair(m, k, n, "int", seed=93, bound=512)
    rows = np.arange(0, m, max(1, m // 60))
    assert np.array_equal(run(bq, A, B)[:, rows], oracle.gemm(A[:, rows], B))


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 8, 12, 13, 16, 17])
@pytest.mark.parametrize("m,k,n", [(5, 3, 7), (66, 130, 33), (17, 64, 18)])
def test_modulus_groups_and_edges(bq, N, m, k, n):
    """Residues are combined four moduli and four columns at a time, split in
    64 x 64 tiles and scaled in groups of 16 rows or columns: counts on and
    beside each edge, odd and even rows (8- and 16-byte accesses), columns
    and rows that are zero, tiny and huge.  Every element
    equals the oracle's."""
    R = inputs.MASKS["real"]
    A, B = inputs.pair(m, k, n, "logspread", seed=92 + N, mask_a=R, mask_b=R)
    A[0, m // 2] = 0.0
    A[0, m - 1] *= 2.0 ** -500
    B[0, :, n // 2] = 0.0
    B[0, :, 0] *= 2.0 ** 300
    print(f"crt edges {m}x{k}x{n} N={N}", flush=True)
    if ozaki2.bits_for(N, k) < 1:
        pytest.skip("too few moduli for this inner dimension")
    got = run(bq, A, B, N, mask_a=R, mask_b=R)
    assert np.array_equal(got[0], ozaki2.product(A[0], B[0], N))


@pytest.mark.parametrize("opA,opB", [("N", "N"), ("T", "T")])
@pytest.mark.parametrize("k", [1024, 2047, 2048, 2050, 3073, 5001])
def test_exponents_over_a_long_inner_dimension(bq, k, opA, opB):
    """Few rows and columns and a long inner dimension: the exponents are
    formed in chunks of it, from 2048 elements on.  Rows and columns whose
    largest element is the first or last of all, or lies on either side of a
    chunk's edge, a zero row and column, denormal and huge ones; few moduli, so
    that the rounding shows every exponent.  Every element equals the
    oracle's."""
    m, n, N = 17, 7, 6
    A, B = inputs.pair(m, k, n, "uniform", seed=95 + k)
    A, B = A * 1e-3, B * 1e-3
    for r, c in enumerate((0, k - 1, 511, 512, 1023, min(1024, k - 1), k // 2)):
        A[0, r, c] = 0.9
        B[0, (k - 1 - c), r] = -0.9
    A[0, 7] = 0.0
    A[0, 8] *= 2.0 ** -1060
    A[0, 9] *= 2.0 ** 400
    B[0, :, 3] = 0.0
    R = inputs.MASKS["real"]
    for c in range(1, 8):
        A[c] = B[c] = 0.0
    print(f"crt exponents k={k} {opA}{opB}", flush=True)
    stored = [np.ascontiguousarray(X.transpose(0, 2, 1)) if op == "T" else X for X, op in ((A, opA), (B, opB))]
    got = run(bq, *stored, N, mask_a=R, mask_b=R, opA=opA, opB=opB)
    assert np.array_equal(got[0], ozaki2.product(A[0], B[0], N))
    A[0, 4, k - 2] = np.nan
    A[0, 5, 1] = np.inf
    got = run(bq, A, B, N, mask_a=R, mask_b=R)[0]
    assert np.all(np.isnan(got[4:6])) and np.all(np.isfinite(np.delete(got, (4, 5), axis=0)))


def test_a_long_inner_dimension_is_shared_by_blocks(bq):
    """The exponents of 16 rows and 16 columns of 131072 elements: 34 MB, read
    by many blocks (a block alone takes about 1 ms)."""
    import torch

    A = torch.rand((8, 16, 131072), dtype=torch.float64, device="cuda")
    B = torch.rand((8, 131072, 16), dtype=torch.float64, device="cuda")
    R = inputs.MASKS["real"]
    for _ in range(2):
        bq.bq_gemm(A, B, prec=PREC, mask_a=R, mask_b=R)
    torch.cuda.synchronize()
    bq.trace_enable(True)
    for _ in range(5):
        bq.bq_gemm(A, B, prec=PREC, mask_a=R, mask_b=R)
    recs = [r for r in bq.trace_read() if r["kernel"] == "split"]
    bq.trace_enable(False)
    us = min(r["ms"] for r in recs[::2]) * 1e3  # exponents, residues in turn
    print(f"exponents of 16 x 131072 and 131072 x 16: {us:.0f} us", flush=True)
    assert len(recs) == 10 and us < 250.0


def test_few_columns_reconstruct_in_few_waves(bq):
    """20000 rows of 16 columns: a block of the reconstruction takes 1024
    columns of one row, so three of its four waves have none and end at once
    (0.66 ms for the eight launches of a product, 1.75 with all four at
    work)."""
    import torch

    A = torch.rand((8, 20000, 64), dtype=torch.float64, device="cuda")
    B = torch.rand((8, 64, 16), dtype=torch.float64, device="cuda")
    C = bq.bq_gemm(A, B, prec=PREC)
    torch.cuda.synchronize()
    rows = torch.tensor([0, 1, 9999, 19999], device="cuda")
    ref = oracle.gemm(A[:, rows].cpu().numpy(), B.cpu().numpy())
    assert oracle.rel_frobenius(C[:, rows].cpu().numpy(), ref) <= TOL
    bq.trace_enable(True)
    for _ in range(5):
        bq.bq_gemm(A, B, prec=PREC)
    ms = [r["ms"] for r in bq.trace_read() if r["kernel"] == "crt_combine"]
    bq.trace_enable(False)
    total = sum(min(ms[q::8]) for q in range(8))
    print(f"reconstruction of 20000 x 16: {total:.2f} ms", flush=True)
    assert len(ms) == 40 and total < 1.2


def test_chunked_exponents_in_a_captured_graph(bq):
    """The exponents of a long inner dimension are cleared and joined by the
    launches of every replay: operands that change between replays, smaller
    ones after larger."""
    import torch

    m, k, n = 20, 4100, 30
    A, B = (torch.from_numpy(X).to("cuda") for X in inputs.pair(m, k, n, "normal", seed=97))
    C = torch.empty((8, m, n), dtype=torch.float64, device="cuda")
    ws = torch.empty(bq.workspace_size(m, n, k, prec=PREC)[0], dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    print(f"capture crt {m}x{k}x{n}", flush=True)
    with torch.cuda.stream(s):
        g.capture_begin(capture_error_mode="thread_local")
        bq.bq_gemm(A, B, C, prec=PREC, workspace=ws, stream=s)
        g.capture_end()
    torch.cuda.synchronize()
    for scale in (1.0, 2.0 ** 40, 2.0 ** -90):
        A.mul_(scale)
        C.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        eager = bq.bq_gemm(A, B, prec=PREC)
        torch.cuda.synchronize()
        assert torch.equal(C, eager), scale
        assert oracle.rel_frobenius(C.cpu().numpy(), oracle.gemm(A.cpu().numpy(), B.cpu().numpy())) <= TOL
    del g


@pytest.mark.parametrize("opA,opB", [("N", "N"), ("N", "T"), ("T", "N")])
@pytest.mark.parametrize("m,k,n", [(5, 3, 7), (64, 128, 64), (130, 190, 66), (200, 257, 190), (400, 300, 350)])
@pytest.mark.parametrize("N", [5, 13, 16, 20])
def test_residues_in_parts(bq, N, m, k, n, opA, opB):
    """Launches of 4 to 240 blocks form the residues in 15 parts to one, with
    more, fewer and as many moduli as parts: a real product equals the oracle's
    in every element."""
    R = inputs.MASKS["real"]
    A, B = inputs.pair(m, k, n, "logspread", seed=98 + N, mask_a=R, mask_b=R)
    if m * n > 20000:
        A[0, 10:] = np.round(A[0, 10:])  # the rest of the rows is not compared
    print(f"crt residues in parts {m}x{k}x{n} N={N} {opA}{opB}", flush=True)
    stored = [np.ascontiguousarray(X.transpose(0, 2, 1)) if op == "T" else X for X, op in ((A, opA), (B, opB))]
    got = run(bq, *stored, N, mask_a=R, mask_b=R, opA=opA, opB=opB)[0]
    rows = slice(0, 10) if m * n > 20000 else slice(0, m)
    assert np.array_equal(got[rows], ozaki2.product(A[0, rows], B[0], N))


def test_small_residue_launches_are_short(bq):
    """The residues of a real product of n = 64 in 15 parts: as long as the
    exponents before them (6 us between trace events; 10.4 in one part)."""
    import torch

    A, B = (torch.rand((8, 64, 64), dtype=torch.float64, device="cuda") for _ in range(2))
    R = inputs.MASKS["real"]
    for _ in range(3):
        bq.bq_gemm(A, B, prec=PREC, mask_a=R, mask_b=R)
    torch.cuda.synchronize()
    bq.trace_enable(True)
    for _ in range(20):
        bq.bq_gemm(A, B, prec=PREC, mask_a=R, mask_b=R)
    recs = [r for r in bq.trace_read() if r["kernel"] == "split"]
    bq.trace_enable(False)
    us = [min(r["ms"] for r in recs[q::2]) * 1e3 for q in (0, 1)]
    print(f"n = 64: exponents {us[0]:.1f} us, residues {us[1]:.1f} us", flush=True)
    assert us[1] < 1.35 * us[0]
