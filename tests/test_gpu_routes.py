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
