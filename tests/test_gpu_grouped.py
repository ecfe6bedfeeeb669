"""Batched form (grouped plans) on the GPU through the C-ABI.

Every product of a batch is checked against the oracle (whole product for
small sizes, sampled rows/columns including the last ones for large ones)
and against the single-call result; graph replays, both work schedules,
workspace re-binding and the split form are covered.
"""
import numpy as np
import pytest

import oracle
from paper_2609_02081_amd import inputs

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_02081_amd as bq

    bq.lib()
    return bq


def _batch(sizes, seed, dist="uniform"):
    import torch

    rng = np.random.default_rng(seed)
    probs = []
    for (m, k, n) in sizes:
        A = torch.from_numpy(inputs.blocks(rng, m, k, dist)).to("cuda")
        B = torch.from_numpy(inputs.blocks(rng, k, n, dist)).to("cuda")
        C = torch.full((8, m, n), float("nan"), dtype=torch.float64, device="cuda")
        probs.append((A, B, C))
    return probs


SMALL = [(17, 33, 65), (64, 64, 64), (130, 70, 129), (1, 5, 1), (200, 150, 90), (96, 200, 33),
         (65, 65, 65), (128, 1, 128), (31, 257, 40), (150, 150, 150), (7, 300, 9), (100, 64, 200)]


def test_small_batch_matches_oracle_and_single_calls(bq):
    import torch

    probs = _batch(SMALL, 61)
    plan = bq.GroupedPlan(probs)
    info = plan.info()
    print(f"grouped small batch: {info}", flush=True)
    plan.launch()
    torch.cuda.synchronize()
    for (A, B, C), shape in zip(probs, SMALL):
        a, b, c = A.cpu().numpy(), B.cpu().numpy(), C.cpu().numpy()
        assert oracle.rel_frobenius(c, oracle.gemm(a, b)) <= TOL, shape
        single = bq.bq_gemm(A, B)
        torch.cuda.synchronize()
        assert oracle.rel_frobenius(c, single.cpu().numpy()) <= 1e-15, shape
    plan.close()


OP_FN = {"N": lambda M: M, "T": oracle.transpose, "C": oracle.conj, "H": oracle.herm}


@pytest.mark.parametrize("prec", ["fp64", "split_int8_crt"])
def test_mixed_ops_batch(bq, prec):
    """All 16 op pairs in one plan, one per problem (T and H read the
    stored matrices: A stored k x m, B stored n x k), ragged shapes: each
    product against the oracle and against the single call."""
    import torch

    rng = np.random.default_rng(62)
    pairs = [(a, b) for a in "NTCH" for b in "NTCH"]
    probs, shapes = [], []
    for idx, (oa, ob) in enumerate(pairs):
        m, k, n = SMALL[idx % len(SMALL)]
        A = torch.from_numpy(inputs.blocks(rng, *((k, m) if oa in "TH" else (m, k)))).to("cuda")
        B = torch.from_numpy(inputs.blocks(rng, *((n, k) if ob in "TH" else (k, n)))).to("cuda")
        C = torch.full((8, m, n), float("nan"), dtype=torch.float64, device="cuda")
        probs.append((A, B, C, oa, ob))
        shapes.append((m, k, n))
    plan = bq.GroupedPlan(probs, prec=prec)
    plan.launch()
    torch.cuda.synchronize()
    for (A, B, C, oa, ob), shape in zip(probs, shapes):
        ref = oracle.gemm(OP_FN[oa](A.cpu().numpy()), OP_FN[ob](B.cpu().numpy()))
        assert oracle.rel_frobenius(C.cpu().numpy(), ref) <= TOL, (oa, ob, shape)
        single = bq.bq_gemm(A, B, opA=oa, opB=ob, prec=prec)
        torch.cuda.synchronize()
        assert oracle.rel_frobenius(C.cpu().numpy(), single.cpu().numpy()) <= 1e-15, (oa, ob, shape)
    plan.close()


def test_replays_identical_with_eager_work_between(bq):
    import torch

    probs = _batch(SMALL[:6], 62)
    plan = bq.GroupedPlan(probs)
    plan.launch()
    torch.cuda.synchronize()
    first = [C.cpu().numpy().copy() for (_, _, C) in probs]
    x = torch.randn(512, 512, dtype=torch.float64, device="cuda")
    for rep in range(3):
        for (_, _, C) in probs:
            C.fill_(float("nan"))
        y = (x @ x).sum()  # unrelated eager work between replays
        plan.launch()
        torch.cuda.synchronize()
        assert torch.isfinite(y).item()
        for f, (_, _, C) in zip(first, probs):
            assert np.array_equal(C.cpu().numpy(), f), rep
    plan.close()


def test_autotune_both_schedules_and_rebind(bq, tmp_path, monkeypatch):
    import torch

    monkeypatch.setenv("BQ_TUNE_CACHE", str(tmp_path / "tune.txt"))
    probs = _batch(SMALL, 63)
    plan = bq.GroupedPlan(probs)
    plan.launch()
    torch.cuda.synchronize()
    ref = [C.cpu().numpy().copy() for (_, _, C) in probs]
    plan.autotune()
    chosen = plan.info()
    print(f"autotune chose {chosen}", flush=True)
    for (_, _, C) in probs:
        C.fill_(0.0)
    # a different workspace buffer re-records the graph
    ws2 = torch.empty(max(1, plan.workspace_size()), dtype=torch.uint8, device="cuda")
    plan.launch(workspace=ws2)
    torch.cuda.synchronize()
    for r, (_, _, C) in zip(ref, probs):
        assert oracle.rel_frobenius(C.cpu().numpy(), r) <= 1e-15
    plan.close()
    # the cache file now holds the choice; a new plan with the same sizes reads it
    text = (tmp_path / "tune.txt").read_text()
    assert text.strip()
    plan2 = bq.GroupedPlan(probs)
    assert plan2.info()["tile_config"] == chosen["tile_config"]
    assert plan2.info()["dynamic"] == chosen["dynamic"]
    assert plan2.info()["per_product_launches"] == chosen["per_product_launches"]
    plan2.close()


def test_every_schedule_gives_the_same_products(bq, tmp_path, monkeypatch):
    """Every tile configuration and schedule the autotuner chooses from,
    forced through the tune cache (the last entry for a key wins): each
    reads back as chosen and every product equals the default plan's to
    1e-15 (the schedules run the same tile code in the same order)."""
    import torch

    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BQ_TUNE_CACHE", str(cache))
    probs = _batch(SMALL[:7], 64)
    plan = bq.GroupedPlan(probs)
    plan.autotune()
    plan.launch()
    torch.cuda.synchronize()
    ref = [C.cpu().numpy().copy() for (_, _, C) in probs]
    plan.close()
    key = cache.read_text().split()[0]
    for cfg in (0, 6):
        for sched in (0, 1, 2, 3):
            with open(cache, "a") as f:
                f.write(f"{key} {cfg} {sched}\n")
            p2 = bq.GroupedPlan(probs)
            info = p2.info()
            assert (info["tile_config"], info["dynamic"], info["per_product_launches"]) == (cfg, sched & 1, sched >> 1)
            for (_, _, C) in probs:
                C.fill_(float("nan"))
            p2.launch()
            torch.cuda.synchronize()
            for r, (_, _, C), shape in zip(ref, probs, SMALL):
                assert oracle.rel_frobenius(C.cpu().numpy(), r) <= 1e-15, (cfg, sched, shape)
            p2.close()


def _sample(n, r, seed):
    rng = np.random.default_rng(seed)
    if n <= r:
        return np.arange(n)
    idx = np.sort(rng.choice(n - 1, size=r - 1, replace=False))
    return np.append(idx, n - 1)


def test_512_products_log_uniform(bq):
    """512 products, sizes log-uniform over 64..1536 (seed 5), uniform[-1,1]."""
    import torch

    sizes = inputs.batch_sizes(512, 64, 1536, seed=5)
    print(f"512 products: total n^3 = {sum(n ** 3 for n in sizes):.3e}", flush=True)
    probs = []
    for i, n in enumerate(sizes):
        A = inputs.device_uniform(n, n, 1000 + 2 * i, "cuda")
        B = inputs.device_uniform(n, n, 1001 + 2 * i, "cuda")
        probs.append((A, B, torch.empty_like(A)))
    plan = bq.GroupedPlan(probs)
    plan.launch()
    torch.cuda.synchronize()
    print("512 products: launched", flush=True)
    worst = 0.0
    for i, ((A, B, C), n) in enumerate(zip(probs, sizes)):
        rows, cols = _sample(n, 16, 7 * i), _sample(n, 16, 7 * i + 1)
        ri, ci = torch.as_tensor(rows, device="cuda"), torch.as_tensor(cols, device="cuda")
        err = oracle.rel_frobenius(C[:, ri][:, :, ci].cpu().numpy(),
                                   oracle.gemm(A[:, ri, :].cpu().numpy(), B[:, :, ci].cpu().numpy()))
        worst = max(worst, err)
    print(f"512 products: worst sampled rel err {worst:.3e}", flush=True)
    assert worst <= TOL
    plan.close()


@pytest.mark.parametrize("prec", ["split_bf16", "split_fp8", "split_int8", "split_int8_crt"])
def test_split_batch(bq, prec):
    import torch

    probs = _batch(SMALL[:8], 64)
    plan = bq.GroupedPlan(probs, prec=prec)
    plan.launch()
    torch.cuda.synchronize()
    for (A, B, C), shape in zip(probs, SMALL):
        err = oracle.rel_frobenius(C.cpu().numpy(), oracle.gemm(A.cpu().numpy(), B.cpu().numpy()))
        assert err <= TOL, (shape, err)
    plan.close()


def test_rejects_overlapping_outputs(bq):
    import torch

    A = torch.rand(8, 32, 32, dtype=torch.float64, device="cuda")
    B = torch.rand(8, 32, 32, dtype=torch.float64, device="cuda")
    C = torch.empty(8, 32, 32, dtype=torch.float64, device="cuda")
    with pytest.raises(bq.BqError) as e:
        bq.GroupedPlan([(A, B, C), (B, A, C)])
    assert e.value.code == 3
    Amask = A.clone()
    with pytest.raises(bq.BqError) as e:
        bq.GroupedPlan([([Amask[0]] + [None] * 7, B, C)])
    assert e.value.code == 2


@pytest.mark.parametrize("oa,ob", [("N", "N"), ("C", "T"), ("H", "C"), ("T", "H")])
def test_uniform_op_batches(bq, oa, ob):
    """Batches whose problems share one op pair run a kernel with that tile
    variant alone; each product against the single call to 1e-15."""
    import torch

    rng = np.random.default_rng(65)
    probs = []
    for (m, k, n) in SMALL[:6]:
        A = torch.from_numpy(inputs.blocks(rng, *((k, m) if oa in "TH" else (m, k)))).to("cuda")
        B = torch.from_numpy(inputs.blocks(rng, *((n, k) if ob in "TH" else (k, n)))).to("cuda")
        C = torch.full((8, m, n), float("nan"), dtype=torch.float64, device="cuda")
        probs.append((A, B, C))
    plan = bq.GroupedPlan(probs, opA=oa, opB=ob)
    plan.launch()
    torch.cuda.synchronize()
    for (A, B, C), shape in zip(probs, SMALL):
        single = bq.bq_gemm(A, B, opA=oa, opB=ob)
        torch.cuda.synchronize()
        assert oracle.rel_frobenius(C.cpu().numpy(), single.cpu().numpy()) <= 1e-15, (oa, ob, shape)
    plan.close()


def _padded(data, pad, torch):
    """(8, rows, cols) device view of `data` inside a buffer with `pad` NaN
    columns after each row (leading dimension cols + pad)."""
    rows, cols = data.shape[1], data.shape[2]
    buf = torch.full((8, rows, cols + pad), float("nan"), dtype=torch.float64, device="cuda")
    buf[:, :, :cols] = torch.from_numpy(data).to("cuda")
    return buf[:, :, :cols]


@pytest.mark.parametrize("oa,ob", [("N", "N"), ("T", "H"), ("H", "N"), ("C", "T")])
def test_padded_operands_with_nan_padding(bq, oa, ob):
    """Operands whose rows are padded (odd and even leading dimensions, odd
    and even stored widths) with NaN in the padding, edge tiles on both
    sides and several full k-steps: the batched tiles read their full
    k-steps without bounds checks, and padding may reach only outputs
    outside the matrix, never stored.  Every product is finite and matches
    the oracle on the unpadded operands and the single call."""
    import torch

    rng = np.random.default_rng(66)
    shapes = [(77, 80, 45), (130, 97, 66), (64, 48, 129), (33, 160, 31), (100, 64, 100), (65, 130, 70)]
    pads = [1, 2, 3, 6, 0, 5]
    probs, refs = [], []
    for (m, k, n), pad in zip(shapes, pads):
        a = inputs.blocks(rng, *((k, m) if oa in "TH" else (m, k)))
        b = inputs.blocks(rng, *((n, k) if ob in "TH" else (k, n)))
        A, B = _padded(a, pad, torch), _padded(b, pad + 1, torch)
        C = torch.full((8, m, n), float("nan"), dtype=torch.float64, device="cuda")
        probs.append((A, B, C))
        refs.append(oracle.gemm(OP_FN[oa](a), OP_FN[ob](b)))
    print(f"padded operands, op {oa}{ob}", flush=True)
    plan = bq.GroupedPlan(probs, opA=oa, opB=ob)
    plan.launch()
    torch.cuda.synchronize()
    for (A, B, C), ref, shape in zip(probs, refs, shapes):
        c = C.cpu().numpy()
        assert np.all(np.isfinite(c)), shape
        assert oracle.rel_frobenius(c, ref) <= TOL, shape
        single = bq.bq_gemm(A, B, opA=oa, opB=ob)
        torch.cuda.synchronize()
        assert oracle.rel_frobenius(c, single.cpu().numpy()) <= 1e-15, shape
    plan.close()


@pytest.mark.parametrize("opA,opB", [("N", "N"), ("H", "T")])
@pytest.mark.parametrize("odd", [0, 1])
def test_one_launch_batches_equal_single_calls(bq, opA, opB, odd):
    """The batched one-launch configuration (13) on small batches, chosen by
    default: 16 x 16 and 32 x 32 tiles, ragged edges, one-element products,
    even and odd leading dimensions.  Tiles run the code of the single call,
    so every product equals it bit for bit."""
    import torch

    shapes = [(1, 1, 1), (16, 16, 16), (33, 40, 31), (100, 90, 80), (257, 64, 130), (400, 33, 390), (64, 300, 64)]
    probs = []
    for i, (m, k, n) in enumerate(shapes):
        def draw(r, c, seed):
            X = inputs.device_uniform(r, c + odd, seed, "cuda")
            return X[:, :, :c]
        A = draw(*((k, m) if opA == "H" else (m, k)), 500 + i)
        B = draw(*((n, k) if opB == "T" else (k, n)), 600 + i)
        probs.append((A, B, torch.full((8, m, n), float("nan"), dtype=torch.float64, device="cuda")))
    print(f"one-launch batch {opA}{opB} odd {odd}", flush=True)
    plan = bq.GroupedPlan(probs, opA=opA, opB=opB)
    assert plan.info()["tile_config"] == 13
    plan.launch()
    torch.cuda.synchronize()
    for (A, B, C), shape in zip(probs, shapes):
        single = bq.bq_gemm(A, B, opA=opA, opB=opB)
        torch.cuda.synchronize()
        assert torch.equal(C, single), shape
    plan.close()


def test_tune_cache_keys(bq, tmp_path, monkeypatch):
    """A cached choice holds for batches that it was made on: the key tells
    even rows from odd ones and plain operands from transposed ones, and an
    entry whose key has sizes alone (written when there were two
    configurations to choose from) leaves the default."""
    import torch

    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BQ_TUNE_CACHE", str(cache))
    n, count = 64, 5

    def problems(pad):
        draw = lambda s: inputs.device_uniform(n, n + pad, s, "cuda")[:, :, :n]
        return [(draw(70 + i), draw(80 + i), torch.empty((8, n, n), dtype=torch.float64, device="cuda"))
                for i in range(count)]

    kinds = [(problems(0), "N", "N"), (problems(1), "N", "N"), (problems(0), "H", "N"), (problems(0), "N", "T")]
    keys = []
    for probs, oa, ob in kinds:
        plan = bq.GroupedPlan(probs, opA=oa, opB=ob)
        default = plan.info()["tile_config"]
        assert default == 13
        plan.autotune()
        plan.close()
        keys.append(cache.read_text().splitlines()[-1].split()[0])
    print(f"tune cache keys: {keys}", flush=True)
    assert len(set(keys)) == len(keys)

    # The choice 0 for the first batch is the first batch's alone.
    cache.write_text(f"{keys[0]} 0 3\n")
    chosen = []
    for probs, oa, ob in kinds:
        plan = bq.GroupedPlan(probs, opA=oa, opB=ob)
        chosen.append(plan.info()["tile_config"])
        plan.close()
    assert chosen == [0, 13, 13, 13]

    # A key of device, precision and sizes: FNV-1a over m, n, k.
    h = 1469598103934665603
    for _ in range(count):
        for x in (n, n, n):
            h = (h ^ x) * 1099511628211 % 2 ** 64
    device = keys[0][keys[0].index("gfx"):].rsplit(":", 1)[0]
    cache.write_text(f"{device}:{h:x} 0 3\n")
    plan = bq.GroupedPlan(kinds[0][0])
    assert plan.info()["tile_config"] == 13
    plan.close()


def test_tables_of_the_configuration_in_use(bq, tmp_path, monkeypatch):
    """A plan holds the item table of the one-launch tiles only once it runs
    them: one product of odd rows, n = 16383, takes configuration 0, whose items
    (nine for each 64 x 64 tile, 16 bytes) are 9.4 MB; the one-launch items would
    be 4.2 MB more.  Small odd batches take 0 by their cache entry and 13 by the
    autotuner afterwards, with the same products."""
    import torch

    n = 16383
    A = torch.empty((8, n, n), dtype=torch.float64, device="cuda")
    C = torch.empty_like(A)
    bq.GroupedPlan(_batch(SMALL[:1], 66)).close()  # the library's own memory, from its first plan on
    torch.cuda.synchronize()
    print(f"plan of one product, n = {n}", flush=True)
    before = torch.cuda.mem_get_info()[0]
    plan = bq.GroupedPlan([(A, A, C)])
    used = before - torch.cuda.mem_get_info()[0]
    assert plan.info()["tile_config"] == 0
    plan.close()
    del A, C
    print(f"{used / 1e6:.1f} MB", flush=True)
    assert used < 14.5e6

    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BQ_TUNE_CACHE", str(cache))
    probs = _batch(SMALL[:4], 67)
    plan = bq.GroupedPlan(probs)
    plan.autotune()
    plan.close()
    key = cache.read_text().split()[0]
    cache.write_text(f"{key} 0 3\n")
    plan = bq.GroupedPlan(probs)
    assert plan.info()["tile_config"] == 0
    plan.launch()
    torch.cuda.synchronize()
    ref = [C.clone() for (_, _, C) in probs]
    cache.write_text(f"{key} 13 0\n")
    other = bq.GroupedPlan(probs)
    assert other.info()["tile_config"] == 13
    for p in (other, plan):
        for (_, _, C) in probs:
            C.fill_(float("nan"))
        if p is plan:
            p.autotune()  # its first use of configuration 13, or a choice among all
        p.launch()
        torch.cuda.synchronize()
        for r, (_, _, C) in zip(ref, probs):
            assert oracle.rel_frobenius(C.cpu().numpy(), r.cpu().numpy()) <= 1e-15
        p.close()


@pytest.mark.parametrize("prec", ["fp64", "split_int8_crt"])
def test_traced_launch_names_the_plans_work_items(bq, prec):
    """The trace record of a launch has the problem count and the work items
    that the plan reports (of the one-launch tiles, where it runs them)."""
    import torch

    probs = _batch(SMALL[:5], 68)
    plan = bq.GroupedPlan(probs, prec=prec)
    info = plan.info()
    plan.launch()
    torch.cuda.synchronize()
    bq.trace_read()
    bq.trace_enable(True)
    plan.launch()
    recs = bq.trace_read()
    bq.trace_enable(False)
    plan.close()
    print(f"{prec}: {info}", flush=True)
    assert [(r["kernel"], r["m"], r["n"]) for r in recs] == [("grouped", len(probs), info["work_items"])]
    if prec == "fp64":
        assert info["tile_config"] == recs[0]["config"] == 13
