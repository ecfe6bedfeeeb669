"""Which kernels a product runs (through the C-ABI, seen in the trace), and that
the routes agree.

FP64 products of all eight (or four real-quaternion) components run either in
one launch or in one launch per complex (real) product; BQ_TILE_CONFIG with a
configuration of their kind selects the latter at any size.  Both take the same
products, sums and additions in the same order, so their results are equal bit
for bit.
"""
import numpy as np
import pytest

import oracle
from paper_2609_02081_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_02081_amd as bq

    bq.lib()
    return bq


def traced(bq, call):
    """The result of call() and the tile configurations of its GEMM launches
    (-1: a one-launch product)."""
    import torch

    torch.cuda.synchronize()
    bq.trace_read()
    bq.trace_enable(True)
    try:
        out = call()
        recs = bq.trace_read()
    finally:
        bq.trace_enable(False)
    return out, [r["config"] for r in recs if r["kernel"].startswith("gemm")]


@pytest.mark.parametrize("value,biquaternion,quaternion", [("", [-1], [-1]), ("0", [0] * 8, [-1]), ("3", [-1], [3] * 8),
                                                           ("11", [-1], [11] * 8), ("14", [14] * 8, [14] * 8),
                                                           ("6", [-1], [-1]), ("13", [-1], [-1])])
def test_tile_configuration_of_a_kind(bq, monkeypatch, value, biquaternion, quaternion):
    """BQ_TILE_CONFIG is heard by the products it suits (complex ones 0 and 14,
    real ones 3, 11 and 14) and by no others."""
    import torch

    monkeypatch.setenv("BQ_TILE_CONFIG", value)
    print(f"BQ_TILE_CONFIG={value}", flush=True)
    for mask, want in ((0xFF, biquaternion), (0x0F, quaternion)):
        A, B = inputs.pair(140, 70, 150, "int", seed=14, bound=512, mask_a=mask, mask_b=mask)
        a, b = torch.from_numpy(A).to("cuda"), torch.from_numpy(B).to("cuda")
        C, configs = traced(bq, lambda: bq.bq_gemm(a, b, mask_a=mask, mask_b=mask))
        assert configs == want, (hex(mask), configs)
        assert np.array_equal(C.cpu().numpy(), oracle.gemm(A, B))


@pytest.mark.parametrize("n,one", [(2301, True), (3001, False)])
def test_large_real_quaternions_with_odd_rows(bq, n, one):
    """Operands of 339 MB run in one launch (3.86 ms against 4.70 in a launch
    for each product), of 576 MB in eight (8.77 against 9.37): past the 256 MB
    cache the 8-byte loads of odd rows take longer."""
    import torch

    A = inputs.device_uniform(n, n, 16, "cuda")[:4]
    B = inputs.device_uniform(n, n, 17, "cuda")[:4]
    C = torch.full((4, n, n), float("nan"), dtype=torch.float64, device="cuda")
    print(f"real quaternions n={n}", flush=True)
    _, configs = traced(bq, lambda: bq.rq_gemm(list(A), list(B), list(C)))
    assert (configs == [-1]) == one, configs
    rows, cols = torch.tensor([0, 1, 1500, n - 1], device="cuda"), torch.tensor([0, 63, 1001, n - 2, n - 1], device="cuda")
    full = [np.concatenate([X.cpu().numpy(), np.zeros(X.shape)]) for X in (A[:, rows], B[:, :, cols])]
    assert oracle.rel_frobenius(np.concatenate([C[:, rows][:, :, cols].cpu().numpy(), np.zeros((4, 4, 5))]),
                                oracle.gemm(*full)) <= 1e-12


@pytest.mark.parametrize("n,opA,opB,one", [(3072, "N", "N", False), (3136, "N", "N", True), (3392, "T", "N", False),
                                           (2501, "T", "N", True), (2501, "N", "T", False)])
def test_large_biquaternions_take_the_shorter_route(bq, n, opA, opB, one):
    """Sizes where the routes lie 4 to 11 % apart (one launch against one for
    each product: n = 3072 23.6 ms against 22.6, 3136 24.5 against 25.4, 3392
    with A transposed 30.1 against 29.0; odd rows, 2501 with A transposed 13.7
    against 15.3, with B transposed 16.9 against 16.0)."""
    import torch

    A = inputs.device_uniform(n, n, 18, "cuda")
    B = inputs.device_uniform(n, n, 19, "cuda")
    print(f"biquaternions n={n} {opA}{opB}", flush=True)
    C, configs = traced(bq, lambda: bq.bq_gemm(A, B, opA=opA, opB=opB))
    assert (configs == [-1]) == one, configs
    rows, cols = torch.tensor([0, 1, 1500, n - 1], device="cuda"), torch.tensor([0, 63, 1001, n - 1], device="cuda")
    a = (A[:, :, rows] if opA == "T" else A[:, rows]).cpu().numpy()
    b = (B[:, cols] if opB == "T" else B[:, :, cols]).cpu().numpy()
    ref = oracle.gemm(oracle.transpose(a) if opA == "T" else a, oracle.transpose(b) if opB == "T" else b)
    assert oracle.rel_frobenius(C[:, rows][:, :, cols].cpu().numpy(), ref) <= 1e-12


@pytest.mark.parametrize("mask,config", [(0xFF, "0"), (0xFF, "14"), (0x0F, "3"), (0x0F, "14")])
@pytest.mark.parametrize("opA,opB", [("N", "N"), ("H", "N"), ("C", "T"), ("T", "H")])
def test_one_launch_equals_one_per_product(bq, monkeypatch, mask, config, opA, opB):
    """Random FP64 inputs of very different magnitudes, odd and even rows, one
    tile to several hundred, ragged k: the two routes give the same bits."""
    import torch

    for i, (m, k, n, pad) in enumerate([(1, 1, 1, 0), (17, 31, 33, 1), (64, 64, 64, 0), (130, 257, 67, 0),
                                        (300, 100, 290, 1), (640, 40, 650, 0)]):
        rng = np.random.default_rng(300 + i)

        def stored(rows, cols):
            X = torch.full((8, rows, cols + pad), float("nan"), dtype=torch.float64, device="cuda")
            X[:, :, :cols] = torch.from_numpy(inputs.blocks(rng, rows, cols, "logspread")).to("cuda")
            return X[:, :, :cols]

        A = stored(*((k, m) if opA in "TH" else (m, k)))
        B = stored(*((n, k) if opB in "TH" else (k, n)))
        kw = dict(opA=opA, opB=opB, mask_a=mask, mask_b=mask)
        print(f"routes {m}x{k}x{n} pad {pad} {opA}{opB} mask {mask:#x} config {config}", flush=True)
        monkeypatch.delenv("BQ_TILE_CONFIG", raising=False)
        one, c1 = traced(bq, lambda: bq.bq_gemm(A, B, **kw))
        monkeypatch.setenv("BQ_TILE_CONFIG", config)
        per, c8 = traced(bq, lambda: bq.bq_gemm(A, B, **kw))
        streamed, cs = traced(bq, lambda: bq.bq_gemm(A, B, streamed=True, **kw))
        assert c1 == [-1] and c8 == cs == [int(config)] * 8
        assert torch.equal(one, per), (m, k, n)
        assert torch.equal(streamed, per), (m, k, n)


@pytest.mark.parametrize("mask,config", [(0xFF, "0"), (0x0F, "14")])
@pytest.mark.parametrize("scale", [-1072, -1060, -1022])
def test_routes_agree_on_denormals(bq, monkeypatch, mask, config, scale):
    """Products among the denormals, where a quarter of a product of the
    Hadamard part rounds: both routes round it before they add it."""
    import torch

    m, k, n = 45, 30, 50
    A, B = inputs.pair(m, k, n, "normal", seed=15, mask_a=mask, mask_b=mask)
    a, b = torch.from_numpy(A).to("cuda") * 2.0 ** (scale + 1000), torch.from_numpy(B).to("cuda") * 2.0 ** -1000
    a, b = a.contiguous(), b.contiguous()
    print(f"denormal products 2^{scale} mask {mask:#x} config {config}", flush=True)
    monkeypatch.delenv("BQ_TILE_CONFIG", raising=False)
    one, c1 = traced(bq, lambda: bq.bq_gemm(a, b, mask_a=mask, mask_b=mask))
    monkeypatch.setenv("BQ_TILE_CONFIG", config)
    per, c8 = traced(bq, lambda: bq.bq_gemm(a, b, mask_a=mask, mask_b=mask))
    assert c1 == [-1] and c8 == [int(config)] * 8
    assert torch.equal(one, per)
    assert bool((one[:4] != 0).any())


# The tests of the per-product kernels (by function, arguments), which small and
# ordinary products reach with BQ_TILE_CONFIG only.
import test_gpu_capture as capture  # noqa: E402
import test_gpu_grouped as grouped  # noqa: E402
import test_gpu_parity as parity  # noqa: E402
import test_zz_no_alloc as noalloc  # noqa: E402

OPS = [(a, b) for a in "NTCH" for b in "NTCH"]
SMALL_PRODUCTS = [
    *((parity.test_random_uniform, s) for s in [(256, 256, 256), (1, 1, 1), (130, 257, 67), (200, 16, 300), (64, 1000, 33)]),
    *((parity.test_integer_bit_exact, s) for s in [(64, 64, 64), (70, 50, 45), (129, 96, 130)]),
    *((parity.test_all_ops, s) for s in OPS),
    *((parity.test_transposed_ops_integer_bit_exact, s) for s in [("T", "N"), ("N", "H"), ("H", "T")]),
    *((parity.test_transposed_ops_streamed_and_masks, s) for s in [("T", "H"), ("H", "N")]),
    (parity.test_transpose_reverses_products, ()),
    (parity.test_streamed_equals_resident, ()),
    (parity.test_side_stream, ()),
    (parity.test_guard_band_untouched, ()),
    (parity.test_nan_row_propagation, ()),
    (noalloc.test_two_calls_second_smaller, ()),
]
LARGE_PRODUCTS = [
    *(("0", parity.test_two_deep_with_edge_tiles, s) for s in [(2050, 1030, 2060), (2047, 1041, 2049)]),
    *(("0", parity.test_large_products_odd_and_ragged_k, (k, 0xFF)) for k in (1040, 1031, 1024)),
    *(("11", parity.test_real_products_in_large_blocks, (*s, 0x0F))
      for s in [(2040, 1001, 2040), (4100, 96, 4100), (2048, 33, 2056)]),
    ("0", noalloc.test_streamed_plan_and_split_form, ()),
]


def _name(x):
    return x.__name__ if callable(x) else str(x)


def _run_forced(bq, monkeypatch, config, test, args):
    monkeypatch.setenv("BQ_TILE_CONFIG", config)
    _, configs = traced(bq, lambda: test(bq, *args))
    assert int(config) in configs, set(configs)
    if config in ("0", "14"):
        assert -1 not in configs or test is parity.test_transposed_ops_streamed_and_masks  # its mask is a real one


@pytest.mark.parametrize("config", ["0", "14"])
@pytest.mark.parametrize("test,args", SMALL_PRODUCTS, ids=_name)
def test_small_products_in_a_launch_each(bq, monkeypatch, config, test, args):
    """64 x 64 and 32 x 32 tiles of the complex products, resident and
    streamed, plain and transposed loads, edge tiles, NaN, a side stream."""
    _run_forced(bq, monkeypatch, config, test, args)


@pytest.mark.parametrize("config,test,args", LARGE_PRODUCTS, ids=_name)
def test_large_products_in_a_launch_each(bq, monkeypatch, config, test, args):
    """The two-deep pipeline with and without edge tiles, 128 x 128 blocks of
    real-quaternion products, the streamed plan of bq_gemm_noalloc."""
    _run_forced(bq, monkeypatch, config, test, args)


@pytest.mark.parametrize("order", ["0,4", "1,1", "1,16"])
@pytest.mark.parametrize("config", ["0", "14"])
def test_tile_orders_of_a_launch_each(bq, monkeypatch, config, order):
    monkeypatch.setenv("BQ_TILE_ORDER", order)
    _run_forced(bq, monkeypatch, config, parity.test_integer_bit_exact, (330, 200, 270))


@pytest.mark.parametrize("entry", ["bq_gemm", "bq_gemm_noalloc"])
@pytest.mark.parametrize("config", ["0", "14"])
def test_captured_launches_of_each_product(bq, monkeypatch, config, entry):
    """Ten launches in a captured graph, replayed with eager work between."""
    monkeypatch.setenv("BQ_TILE_CONFIG", config)
    capture.test_captured_product_replays(bq, entry)


@pytest.mark.parametrize("cfg,schedule", [(0, 3), (0, 0), (6, 2), (6, 1), (13, 0)])
@pytest.mark.parametrize("test,args", [(grouped.test_small_batch_matches_oracle_and_single_calls, ()),
                                       (grouped.test_mixed_ops_batch, ("fp64",)),
                                       (grouped.test_replays_identical_with_eager_work_between, ()),
                                       *((grouped.test_uniform_op_batches, s)
                                         for s in [("N", "N"), ("C", "T"), ("H", "C"), ("T", "H")]),
                                       *((grouped.test_padded_operands_with_nan_padding, s)
                                         for s in [("N", "N"), ("T", "H"), ("H", "N"), ("C", "T")])], ids=_name)
def test_batches_in_every_configuration(bq, monkeypatch, tmp_path, test, args, cfg, schedule):
    """Each configuration and schedule of a batched plan on batches that run
    in one launch by default: mixed and uniform ops, NaN in the padding."""
    _force_plans(bq, monkeypatch, tmp_path, cfg, schedule)
    test(bq, *args)


def _force_plans(bq, monkeypatch, tmp_path, cfg, schedule):
    """Plans made by bq.GroupedPlan take the configuration through the tune
    cache (the last entry of a key wins)."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BQ_TUNE_CACHE", str(cache))
    Plan = bq.GroupedPlan

    def make(problems, **kw):
        p = Plan(problems, **kw)
        p.autotune()
        p.close()
        for prob in problems:
            prob[2].fill_(float("nan"))
        key = cache.read_text().splitlines()[-1].split()[0]
        with open(cache, "a") as f:
            f.write(f"{key} {cfg} {schedule}\n")
        p = Plan(problems, **kw)
        info = p.info()
        assert (info["tile_config"], info["dynamic"], info["per_product_launches"]) == (cfg, schedule & 1, schedule >> 1)
        return p

    monkeypatch.setattr(bq, "GroupedPlan", make)


def _far_rows(rng, rows, cols, ld, torch):
    """Eight components (rows x cols) in one buffer, their rows ld apart."""
    X = inputs.blocks(rng, rows, cols, "uniform")
    buf = torch.zeros((rows, ld), dtype=torch.float64, device="cuda")
    comps = [buf[:, 64 * c:64 * c + cols] for c in range(8)]
    for c in range(8):
        comps[c].copy_(torch.from_numpy(X[c]))
    return X, comps


@pytest.mark.parametrize("opA,opB", [("N", "N"), ("T", "N"), ("N", "T"), ("T", "T")])
@pytest.mark.parametrize("ld", [4_500_000, 8_388_592, 9_000_000])
def test_rows_far_apart(bq, monkeypatch, tmp_path, ld, opA, opB):
    """Rows 4.5e6, 8388592 and 9e6 doubles apart, single calls and batched
    plans.  A tile of 32 rows spans 2^31 bytes from 8388607 on, so the first two
    run in one launch, the second with offsets up to the last that buffer loads
    reach, and the third in a launch for each product; 64 rows span as much from
    4.2e6 on, so that operands stored along k reach the kernels with pointer
    loads in all three where 64 x 64 tiles are asked for.  38 rows and 35 columns
    (two tiles of 32, the second short), against the oracle."""
    import torch

    m, k, n = 38, 40, 35
    rng = np.random.default_rng(81)
    a, A = _far_rows(rng, *((k, m) if opA == "T" else (m, k)), ld, torch)
    b, B = _far_rows(rng, *((n, k) if opB == "T" else (k, n)), ld, torch)
    ref = oracle.gemm(oracle.transpose(a) if opA == "T" else a, oracle.transpose(b) if opB == "T" else b)
    one = ld < 8_388_607
    print(f"rows {ld} apart, {opA}{opB}: single calls", flush=True)
    C, configs = traced(bq, lambda: bq.bq_gemm(A, B, opA=opA, opB=opB))
    assert configs == ([-1] if one else [14] * 8)
    assert oracle.rel_frobenius(C.cpu().numpy(), ref) <= 1e-12
    monkeypatch.setenv("BQ_TILE_CONFIG", "0")
    C, configs = traced(bq, lambda: bq.bq_gemm(A, B, opA=opA, opB=opB))
    assert configs == [0] * 8
    assert oracle.rel_frobenius(C.cpu().numpy(), ref) <= 1e-12
    print("batched plans", flush=True)
    C.fill_(float("nan"))
    plan = bq.GroupedPlan([(A, B, C)], opA=opA, opB=opB)
    assert (plan.info()["tile_config"] == 13) == one
    plan.launch()
    torch.cuda.synchronize()
    assert oracle.rel_frobenius(C.cpu().numpy(), ref) <= 1e-12
    plan.close()
    for cfg in (0, 6):
        with monkeypatch.context() as mp:
            _force_plans(bq, mp, tmp_path, cfg, 3)
            plan = bq.GroupedPlan([(A, B, C)], opA=opA, opB=opB)
        plan.launch()
        torch.cuda.synchronize()
        assert oracle.rel_frobenius(C.cpu().numpy(), ref) <= 1e-12
        plan.close()
