"""Parity of the three top-k states with the CPU oracle, bit for bit, through the C ABI.

The selection is unique under the tie rule (lower index wins) and the output order is fixed
(increasing index), so indices and values are compared exactly.
"""
import json
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2605_28213_amd import gemm, topk
from paper_2605_28213_amd import inputs as gen

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT_DIR = os.environ.get("GEMM_GATE_OUT") or os.path.join(ROOT, "gate_out")


def run_state(variant, x, n, k, *, offset_bytes=0):
    """x: (batch, ld) fp32 numpy buffer.  Returns (status, idx, val, query)."""
    batch, ld = x.shape
    raw = torch.empty(x.size * 4 + 64, dtype=torch.uint8, device="cuda")
    dx = raw[offset_bytes:offset_bytes + x.size * 4]
    dx.copy_(torch.from_numpy(x.reshape(-1).view(np.uint8)))
    didx = torch.full((batch * max(k, 1),), -7, dtype=torch.int32, device="cuda")
    dval = torch.full((batch * max(k, 1),), -7.0, dtype=torch.float32, device="cuda")
    d = topk.make_desc(batch, n, k, ld=ld)
    q = topk.topk_query(variant, d, dx)
    rc = topk.topk_run(variant, d, dx, didx, dval)
    torch.cuda.synchronize()
    return rc, didx.cpu().numpy()[: batch * k].reshape(batch, k), dval.cpu().numpy()[: batch * k].reshape(batch, k), q


def check(variant, x, n, k):
    rc, idx, val, q = run_state(variant, x, n, k)
    assert rc == gemm.GEMM_OK, (gemm.gemm_status_string(rc), topk.topk_last_launch_error(), q)
    ridx, rval = oracle.topk(x[:, :n], k)
    np.testing.assert_array_equal(idx, ridx)
    np.testing.assert_array_equal(val.view(np.uint32), rval.view(np.uint32))


@pytest.mark.parametrize("name", ["TOPK", "TOPK_ties", "TOPK_small", "TOPK_ragged", "TOPK_wide", "TOPK_long"])
@pytest.mark.parametrize("variant", [0, 1, 2])
def test_every_state_matches_the_oracle_bit_for_bit(name, variant):
    cfg = gen.TOPK_CONFIGS[name]
    for seed in (0, 1, 2):
        x = gen.make_topk_inputs(cfg, seed)
        if (variant == 0 and cfg.n > 65536) or (variant == 2 and cfg.n > 16384):
            rc, idx, val, q = run_state(variant, x, cfg.n, cfg.k)
            assert rc == gemm.GEMM_ERR_PRECONDITION and q.violated != 0
            assert (idx == -7).all()                    # nothing was launched
            continue
        if variant == 0 and cfg.k > 1024 and seed > 0:
            continue                                    # k rounds each: one seed is enough for the slow state
        check(variant, x, cfg.n, cfg.k)


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("n,k", [(1, 1), (2, 1), (4, 4), (63, 7), (64, 64), (65, 1), (257, 256), (1000, 1), (4096, 4096), (4100, 17)])
def test_edge_sizes(variant, n, k):
    rng = np.random.default_rng(n * 1000 + k)
    ld = (n + 3) // 4 * 4
    x = rng.standard_normal((3, ld)).astype(np.float32)
    x[:, n:] = 1e30
    check(variant, x, n, k)


@pytest.mark.parametrize("variant", [0, 1, 2])
def test_degenerate_values(variant):
    n = 512
    rows = [np.full(n, 3.0, np.float32),                                    # all equal: the first k indices
            np.zeros(n, np.float32),
            np.where(np.arange(n) % 2 == 0, -0.0, 0.0).astype(np.float32),  # signed zeros tie
            np.arange(n, dtype=np.float32), np.arange(n, dtype=np.float32)[::-1].copy(),
            np.where(np.arange(n) % 3 == 0, np.inf, -np.inf).astype(np.float32),
            np.concatenate([np.full(n // 2, -1e38, np.float32), np.full(n // 2, 1e-45, np.float32)]),   # denormals, huge negatives
            -np.abs(np.random.default_rng(5).standard_normal(n)).astype(np.float32)]                    # all negative
    x = np.stack(rows)
    for k in (1, 100, 171, 511, 512):
        check(variant, x, n, k)


def test_long_runs_of_equal_values_in_long_rows():
    """More than 32767 elements equal to the threshold in a row shorter than 65536 (the compaction's
    counts share one word there), and a row beyond 65536 (two scans)."""
    for n, k in ((50000, 40000), (65535, 65000), (66000, 40000)):
        x = np.full((2, n), 1.5, np.float32)
        x[1, ::7] = 2.0
        x[1, 5::11] = -3.0
        check(1, x, n, k)


def test_empty_calls_and_misaligned_rows():
    x = np.random.default_rng(0).standard_normal((2, 64)).astype(np.float32)
    for variant in range(3):
        rc, idx, val, q = run_state(variant, x, 64, 0)
        assert rc == gemm.GEMM_OK and q.grid == 0
    rc, idx, val, q = run_state(2, x, 64, 8, offset_bytes=4)                 # x not 16-byte aligned: the resident state refuses
    assert rc == gemm.GEMM_ERR_PRECONDITION and topk.Query.names(q.violated) == ["ALIGN16"]
    rc, idx, val, q = run_state(1, x, 64, 8, offset_bytes=4)                 # the streaming state does not care
    assert rc == gemm.GEMM_OK
    ridx, rval = oracle.topk(x, 8)
    np.testing.assert_array_equal(idx, ridx)


def test_gate_table_of_the_paper_shape():
    cfg = gen.TOPK_CONFIGS["TOPK"]
    x = gen.make_topk_inputs(cfg, 0)
    dx = torch.from_numpy(x).cuda()
    didx = torch.empty(cfg.batch * cfg.k, dtype=torch.int32, device="cuda")
    dval = torch.empty(cfg.batch * cfg.k, dtype=torch.float32, device="cuda")
    d = topk.make_desc(cfg.batch, cfg.n, cfg.k)
    rows = []
    for variant in range(3):
        reps = 20 if variant == 0 else 100
        for _ in range(5 if variant == 0 else 25):
            assert topk.topk_run(variant, d, dx, didx, dval) == gemm.GEMM_OK
        torch.cuda.synchronize()
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(reps)]
        for e0, e1 in ev:
            e0.record()
            topk.topk_run(variant, d, dx, didx, dval)
            e1.record()
        torch.cuda.synchronize()
        ts = sorted(e0.elapsed_time(e1) * 1e3 for e0, e1 in ev)
        rows.append({"state": topk.topk_variant_name(variant), "path": topk.topk_query(variant, d, dx).path,
                     "median_us": ts[len(ts) // 2], "min_us": ts[0], "launches": reps})
    os.makedirs(OUT_DIR, exist_ok=True)
    with open(os.path.join(OUT_DIR, "topk_gate_table.txt"), "w") as f:
        for r in rows:
            f.write(json.dumps(r) + "\n")
    assert rows[2]["median_us"] < rows[0]["median_us"] and rows[1]["median_us"] < rows[0]["median_us"]


@pytest.mark.parametrize("n,k", [(4097, 1), (12288, 512), (12289, 1), (12289, 2048), (4097, 2048), (4098, 2049), (8191, 64), (32768, 2048), (70003, 4097), (131072, 64), (262147, 700)])
@pytest.mark.parametrize("values", ["normal", "ascending", "few", "zeros", "neginf"])
def test_long_rows(n, k, values):
    """Rows beyond 4096 elements: without the filter (up to 12288) and with it, a list of candidates that suffices, one
    that overflows (equal values) and k beyond the filter; every length modulo 4, every row start modulo 16 bytes (odd ld)."""
    rng = np.random.default_rng(n + k)
    ld = n | 1
    x = rng.standard_normal((3, ld)).astype(np.float32)
    if values == "ascending":
        x.sort(axis=1)
    elif values == "few":
        x = np.round(x * 2) / 2                          # about 15 values, both zeros among them
    elif values == "zeros":
        x = np.where(rng.random((3, ld)) < 0.999, np.float32(0.0), x).astype(np.float32)
    elif values == "neginf":
        x = np.where(rng.random((3, ld)) < 0.995, np.float32(-np.inf), x).astype(np.float32)
    x[:, n:] = 1e30
    rc, idx, val, q = run_state(1, x, n, k)
    assert rc == gemm.GEMM_OK and q.threads == 1024
    # the oracle counts ranks in O(n^2); a stable sort of the negated row is the same selection (one of the oracle's pins)
    ridx = np.sort(np.argsort(-x[:, :n], axis=1, kind="stable")[:, :k], axis=1)
    np.testing.assert_array_equal(idx, ridx)
    np.testing.assert_array_equal(val.view(np.uint32), np.take_along_axis(x, ridx, 1).view(np.uint32))


@pytest.mark.parametrize("b,n,threads", [(512, 4099, 1024), (513, 4099, 256), (513, 5000, 256), (513, 5001, 1024)])
def test_many_long_rows(b, n, threads):
    """Both sides of the lines beyond which many rows keep 256 lanes each, one row in four of tied values."""
    rng = np.random.default_rng(n)
    x = rng.standard_normal((b, n + 1)).astype(np.float32)
    x[::4] = np.round(x[::4])
    rc, idx, val, q = run_state(1, x, n, 300)
    assert rc == gemm.GEMM_OK and q.threads == threads
    ridx = np.sort(np.argsort(-x[:, :n], axis=1, kind="stable")[:, :300], axis=1)
    np.testing.assert_array_equal(idx, ridx)
    np.testing.assert_array_equal(val.view(np.uint32), np.take_along_axis(x, ridx, 1).view(np.uint32))
