"""Property tests of the host-side planner (gemm_query never launches, so no GPU is needed).

For arbitrary valid descriptors: the condition masks are consistent, STRICT turns exactly the calls
with violated conditions into refusals, the reported scratch follows the packed layout, tile and
simplification switches are accepted only where they mean something, and the launch geometry covers
the problem.
"""
import math

import pytest
from hypothesis import given, settings, strategies as st

from paper_2605_28213_amd import gemm

DT = st.sampled_from([gemm.GEMM_F32, gemm.GEMM_BF16, gemm.GEMM_F16, gemm.GEMM_FP8_E4M3])
LAYOUT = st.sampled_from([gemm.GEMM_ROW_MAJOR, gemm.GEMM_COL_MAJOR])
ES = {gemm.GEMM_F32: 4, gemm.GEMM_BF16: 2, gemm.GEMM_F16: 2, gemm.GEMM_FP8_E4M3: 1}


@st.composite
def descriptors(draw):
    M, N, K = draw(st.integers(1, 5000)), draw(st.integers(1, 5000)), draw(st.integers(1, 5000))
    dt = draw(DT)
    la, lb = draw(LAYOUT), draw(LAYOUT)
    out = gemm.GEMM_BF16 if dt == gemm.GEMM_FP8_E4M3 else dt
    pad = draw(st.sampled_from([0, 0, 1, 3, 8, 16]))
    lda = (K if la == gemm.GEMM_ROW_MAJOR else M) + pad
    ldb = (N if lb == gemm.GEMM_ROW_MAJOR else K) + pad
    return dict(M=M, N=N, K=K, dt=dt, out=out, la=la, lb=lb, lda=lda, ldb=ldb, ldc=N + pad, batch=draw(st.integers(1, 4)))


def make(p, **kw):
    return gemm.make_desc(p["M"], p["N"], p["K"], p["dt"], p["out"], p["la"], p["lb"], lda=p["lda"], ldb=p["ldb"],
                          ldc=p["ldc"], batch=p["batch"], **kw)


@settings(max_examples=300, deadline=None)
@given(descriptors(), st.integers(0, 4))
def test_masks_status_and_geometry_are_consistent(p, variant):
    q = gemm.gemm_query(variant, make(p))
    assert q.status in (gemm.GEMM_OK, gemm.GEMM_ERR_PRECONDITION)
    assert q.violated == q.required & ~q.holds
    assert q.status == gemm.GEMM_OK                                     # every violation has a slow path of the same state
    strict = gemm.gemm_query(variant, make(p, flags=gemm.GEMM_FLAG_STRICT))
    assert (strict.status == gemm.GEMM_ERR_PRECONDITION) == (q.violated != 0)
    assert strict.path == q.path and strict.violated == q.violated
    if q.status == gemm.GEMM_OK:
        assert q.path and q.threads in (64, 128, 256, 512) and q.grid >= 1
        if q.bm and q.bn and "stream" not in q.path and "thin" not in q.path:
            assert q.grid >= math.ceil(p["M"] / q.bm) * math.ceil(p["N"] / q.bn) * p["batch"] or "M-tail" in q.path or \
                    ("persistent" in q.path and q.grid == 256)      # (256 workgroups walking several tiles each)
        assert q.lds_bytes <= 160 * 1024


@settings(max_examples=300, deadline=None)
@given(descriptors())
def test_expert_state_paths_and_scratch(p):
    es = ES[p["dt"]]
    q = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p))
    if p["dt"] == gemm.GEMM_F32:
        # fp32 runs its matrix instruction in the masked kernel only: no fast, packed or streaming form, no scratch
        assert q.status == gemm.GEMM_OK and "masked" in q.path and q.workspace_bytes == 0 and q.violated == 0
        assert (q.bm, q.bn) in ((128, 128), (64, 64)) and q.bk == 32
        return
    fast_ok = (p["la"] == gemm.GEMM_ROW_MAJOR and p["lb"] == gemm.GEMM_COL_MAJOR and (p["lda"] * es) % 16 == 0
               and (p["ldb"] * es) % 16 == 0 and (p["batch"] == 1 or ((p["M"] * p["lda"] * es) % 16 == 0 and (p["N"] * p["ldb"] * es) % 16 == 0)))
    kvec, kslab = 16 // es, 128 // es
    cols = 16 if p["M"] <= 16 else 32 if p["M"] <= 32 else 64
    streams = p["M"] <= 16 or (p["M"] <= 96 and math.ceil(p["N"] / cols) * p["batch"] >= 128)
    group_rows = lambda r: 16 if r <= 16 else 32 if r <= 32 else 48 if r <= 48 else 64 if r <= 64 else 96   # rows a form holds
    if fast_ok and streams and p["K"] % kvec == 0:
        assert q.path == "mfma16-stream(small-M)" and q.workspace_bytes == 0
        assert q.bn == cols and q.bm == group_rows(p["M"]) and q.grid == math.ceil(p["N"] / cols) * p["batch"]
    elif (fast_ok and p["K"] % kvec == 0 and p["M"] > p["N"] and p["N"] <= 96
          and (p["N"] <= 16 or math.ceil(p["M"] / (32 if p["N"] <= 32 else 64)) * p["batch"] >= 128)):
        # few columns: the streaming kernel on the transposed product, strips along M
        strip = 16 if p["N"] <= 16 else 32 if p["N"] <= 32 else 64
        assert q.path == "mfma16-stream(small-N)" and q.workspace_bytes == 0
        assert q.bm == strip and q.bn == group_rows(p["N"]) and q.grid == math.ceil(p["M"] / strip) * p["batch"]
    elif fast_ok and p["K"] % kslab == 0:
        assert q.path.startswith("mfma32-direct-to-lds") and q.violated == 0
        # split-K: offered (through workspace_bytes) when the product has few tiles and a long K, taken when scratch is lent
        nslab, tiles = p["K"] // kslab, math.ceil(p["M"] / 128) * math.ceil(p["N"] / 128)
        # a thin row remainder goes to the streaming kernel when that saves a round of 256 tiles of 256 x 256
        t256 = math.ceil(p["M"] / 256) * math.ceil(p["N"] / 256) * p["batch"]
        t128 = math.ceil(p["M"] / 128) * math.ceil(p["N"] / 128) * p["batch"]
        small = math.ceil(t128 / 512) * (8 if es == 1 else 7) < math.ceil(t256 / 256) * 10
        per_row, rows = math.ceil(p["N"] / 256) * p["batch"], p["M"] // 256
        tail = (p["M"] > 256 and 1 <= p["M"] % 256 <= 64 and p["N"] <= 16384 and not small
                and math.ceil(rows * per_row / 256) < math.ceil((rows + 1) * per_row / 256))
        assert ("M-tail" in q.path) == tail
        splits = 1
        if p["batch"] == 1 and p["M"] > 16 and not tail and tiles < 256:
            for s_ in range(2, 9):
                if nslab % s_ == 0 and nslab // s_ >= 16 and tiles * s_ <= 640:
                    splits = s_
        assert q.workspace_bytes == (splits * p["M"] * p["N"] * 4 if splits > 1 else 0)
        assert "splitK" not in q.path
        if splits > 1:
            lent = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=q.workspace_bytes))
            assert lent.status == gemm.GEMM_OK and lent.path == "mfma32-direct-to-lds+splitK(%d)" % splits
            assert lent.grid == q.grid * splits
            small = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=q.workspace_bytes - 1))
            assert small.status == gemm.GEMM_ERR_WORKSPACE
    elif (p["dt"] in (gemm.GEMM_BF16, gemm.GEMM_F16) and p["la"] == gemm.GEMM_ROW_MAJOR and p["lb"] == gemm.GEMM_ROW_MAJOR
          and math.ceil(p["M"] / 256) * math.ceil(p["N"] / 256) * p["batch"] >= 256 and math.ceil(p["K"] / kslab) >= 3
          and p["lda"] * es <= 1 << 22 and p["K"] * p["ldb"] * es < 1 << 31):
        # both operands row-major and at least 256 tiles: the persistent kernel reads them in place, whatever their
        # alignment and K; nothing violated, no scratch asked for or used
        # a thin remainder of rows that would cost a round of tiles goes to the thin kernel (which also reads B in place)
        per_row, rows = math.ceil(p["N"] / 256) * p["batch"], p["M"] // 256
        thin_tail = (p["M"] > 256 and 1 <= p["M"] % 256 <= 64 and p["N"] <= 16384 and rows * per_row >= 256
                     and (p["K"] + 64) * p["ldb"] * 2 < 1 << 31
                     and math.ceil(rows * per_row / 256) < math.ceil((rows + 1) * per_row / 256))
        assert q.path == "mfma32-direct-to-lds(persistent,B-row-major)" + ("+thin(M-tail)" if thin_tail else "")
        assert q.violated == 0 and q.grid == 256
        assert q.workspace_bytes == 0
        lent = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=1 << 30))
        assert lent.status == gemm.GEMM_OK and lent.path == q.path
    elif (p["dt"] in (gemm.GEMM_BF16, gemm.GEMM_F16) and p["la"] == gemm.GEMM_ROW_MAJOR and p["lb"] == gemm.GEMM_ROW_MAJOR
          and p["M"] <= 64 and (p["K"] + 64) * p["ldb"] * 2 < 1 << 31 and p["M"] * p["lda"] * 2 < 1 << 31):
        # at most 64 rows, both operands row-major: the thin kernel reads B once, in place; no scratch, lent or not
        assert q.path == "mfma16-thin(B-row-major)" and q.violated == 0 and q.workspace_bytes == 0
        cols = 64
        assert q.grid == math.ceil(p["N"] / cols) * p["batch"] and q.bn == cols and q.bm >= min(p["M"], 64) and q.threads == 512
        lent = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=1 << 30))
        assert lent.path == q.path
    else:
        kp = math.ceil(p["K"] / kslab) * kslab
        assert q.path.startswith("mfma32-") and "packed" not in q.path
        # an operand that meets the fast kernel's conditions by itself is used in place, the other one is packed
        whole = p["K"] % kslab == 0
        a_ok = (whole and p["la"] == gemm.GEMM_ROW_MAJOR and (p["lda"] * es) % 16 == 0 and p["lda"] * es <= 1 << 22
                and (p["batch"] == 1 or (p["M"] * p["lda"] * es) % 16 == 0))
        b_ok = (whole and p["lb"] == gemm.GEMM_COL_MAJOR and (p["ldb"] * es) % 16 == 0 and p["ldb"] * es <= 1 << 22
                and (p["batch"] == 1 or (p["N"] * p["ldb"] * es) % 16 == 0))
        assert not (a_ok and b_ok)
        assert q.workspace_bytes == p["batch"] * ((0 if a_ok else p["M"]) + (0 if b_ok else p["N"])) * kp * es
        lent = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=q.workspace_bytes))
        tag = "(B)" if a_ok else "(A)" if b_ok else ""
        in_place = lent.path == q.path and q.path.endswith("(direct-to-lds)")       # (with scratch lent as without: the lines have a test of their own)
        assert lent.status == gemm.GEMM_OK and (in_place or lent.path.startswith("mfma32-packed%s+direct-to-lds" % tag))
        assert not in_place or (es == 2 and p["batch"] == 1)
        small = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=q.workspace_bytes - 1))
        assert small.status == gemm.GEMM_ERR_WORKSPACE
        odd = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4100, workspace_bytes=q.workspace_bytes))
        assert odd.status == gemm.GEMM_ERR_WORKSPACE


@settings(max_examples=200, deadline=None)
@given(descriptors(), st.integers(0, 4), st.sampled_from([gemm.GEMM_FLAG_TILE_128, gemm.GEMM_FLAG_TILE_256,
                                                         gemm.GEMM_FLAG_DEOPT_NO_SWIZZLE, gemm.GEMM_FLAG_DEOPT_NO_OVERLAP,
                                                         gemm.GEMM_FLAG_DEOPT_NO_RASTER, gemm.GEMM_FLAG_MFMA_32X32]))
def test_expert_only_switches_are_refused_elsewhere(p, variant, flag):
    plain = gemm.gemm_query(variant, make(p))
    q = gemm.gemm_query(variant, make(p, flags=flag))
    on_fast_kernel = (variant == gemm.GEMM_K4_MFMA and plain.status == gemm.GEMM_OK and plain.path.startswith("mfma32-direct-to-lds")
                      and "B-row-major" not in plain.path)      # (the in-place form has no simplified states: with a switch the masked kernel keeps the product)
    if on_fast_kernel:
        assert q.status == gemm.GEMM_OK
        if flag == gemm.GEMM_FLAG_TILE_128:
            assert (q.bm, q.bn) == (128, 128)
        if flag in (gemm.GEMM_FLAG_TILE_256, gemm.GEMM_FLAG_DEOPT_NO_SWIZZLE, gemm.GEMM_FLAG_DEOPT_NO_OVERLAP):
            assert (q.bm, q.bn) == (256, 256)
        if flag == gemm.GEMM_FLAG_DEOPT_NO_RASTER:
            assert (q.bm, q.bn) == (plain.bm, plain.bn) and q.path.endswith("-noraster")     # the tile walk is independent of the tile
    elif plain.status == gemm.GEMM_OK:
        assert q.status == gemm.GEMM_ERR_BAD_ARG


@settings(max_examples=150, deadline=None)
@given(descriptors(), st.integers(0, 4))
def test_vector_load_simplification_belongs_to_k2_and_k3(p, variant):
    q = gemm.gemm_query(variant, make(p, flags=gemm.GEMM_FLAG_DEOPT_NO_VECTOR))
    if variant in (gemm.GEMM_K2_VECTORIZED, gemm.GEMM_K3_PIPELINED):
        assert q.status == gemm.GEMM_OK and q.path == "elementwise-masked(-novec)"
        both = gemm.gemm_query(variant, make(p, flags=gemm.GEMM_FLAG_DEOPT_NO_VECTOR | gemm.GEMM_FLAG_DEOPT_NO_RASTER))
        assert both.status == gemm.GEMM_ERR_BAD_ARG
    else:
        assert q.status == gemm.GEMM_ERR_BAD_ARG


ROW, COL = gemm.GEMM_ROW_MAJOR, gemm.GEMM_COL_MAJOR
IN_PLACE_LINES = [  # (M, N, K, layouts, multiple of elements that leading dimensions are odd multiples of, in place)
    (1024, 1024, 20000, ROW, ROW, 1, True), (1024, 1024, 20000, COL, COL, 8, True),         # one 64-tile per CU: always (measured 0.72, 0.64 of packed)
    (1040, 1040, 20000, ROW, ROW, 1, False),
    (2600, 2600, 1900, ROW, COL, 8, True), (2600, 2600, 1940, ROW, COL, 8, False),          # K contiguous in both: 13, 10, 5, 3 x 10^9
    (2000, 2000, 2490, ROW, COL, 4, True), (2000, 2000, 2510, ROW, COL, 4, False),
    (2000, 2000, 1240, ROW, COL, 2, True), (2000, 2000, 1260, ROW, COL, 2, False),
    (2000, 2000, 740, ROW, COL, 1, True), (2000, 2000, 760, ROW, COL, 1, False),
    (2048, 2048, 4096, COL, ROW, 8, True), (2900, 2900, 2960, COL, ROW, 8, True), (2900, 2900, 2980, COL, ROW, 8, False),
    (2000, 2000, 3990, ROW, ROW, 4, True), (2000, 2000, 4010, ROW, ROW, 4, False),          # other layouts: 25, 16, 13, 8
    (2000, 2000, 3240, COL, COL, 2, True), (2000, 2000, 3260, COL, COL, 2, False),
    (2000, 2000, 1990, COL, ROW, 1, True), (2000, 2000, 2010, COL, ROW, 1, False),
    (1400, 1400, 4800, COL, ROW, 1, False), (1200, 1400, 4800, COL, ROW, 4, True), (2000, 1900, 6400, COL, ROW, 8, True),   # long K
    (1200, 1290, 6408, COL, ROW, 8, True), (1300, 1290, 6408, COL, ROW, 8, False),
    (1200, 1000, 5000, ROW, ROW, 4, True), (1300, 1000, 5000, ROW, ROW, 4, False),
    (4096, 1000, 2432, ROW, ROW, 8, True), (4096, 1000, 2496, ROW, ROW, 8, False),          # B alone is packed, A has four times its rows: 10
    (64, 16384, 512, COL, COL, 8, True), (64, 16384, 1024, COL, COL, 8, False),             # A alone, B has 256 times: 0.6
]


def test_packed_or_in_place_by_size_layout_and_alignment():
    """With scratch lent the operands are multiplied where they lie on the side of each line where that is faster."""
    for dt in (gemm.GEMM_BF16, gemm.GEMM_F16):
        for (M, N, K, la, lb, al, in_place) in IN_PLACE_LINES:
            ld = lambda x: next(y for y in range(x, x + 17) if y % (2 * al if al < 8 else 8) == (al if al < 8 else 0))
            p = dict(M=M, N=N, K=K, dt=dt, out=dt, la=la, lb=lb, lda=ld(K if la == ROW else M), ldb=ld(N if lb == ROW else K), ldc=N, batch=1)
            need = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p)).workspace_bytes
            assert need > 0 and gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p)).path.endswith("(direct-to-lds)")
            q = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=need))
            assert q.status == gemm.GEMM_OK and q.path.endswith("(direct-to-lds)") == in_place and ("packed" in q.path) != in_place, (M, N, K, la, lb, al, q.path)
    # an operand's address counts as its rows do
    p = dict(M=2000, N=2000, K=2400, dt=gemm.GEMM_BF16, out=gemm.GEMM_BF16, la=COL, lb=ROW, lda=2000, ldb=2000, ldc=2000, batch=1)
    need = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p)).workspace_bytes
    for A, B, in_place in [(4096, 4096, True), (4098, 4096, False), (4096, 4098, False), (4100, 4096, True)]:
        q = gemm.gemm_query(gemm.GEMM_K4_MFMA, make(p, workspace=4096, workspace_bytes=need), A, B)
        assert q.path.endswith("(direct-to-lds)") == in_place and ("packed" in q.path) != in_place, (A, B, q.path)


def test_which_k_ranges_run_with_a_rotated_walk():
    """One row of 128-tiles and a B of at least 192 MiB, more than the Infinity Cache keeps from pass to pass."""
    for (dt, M, N, K, path) in [(gemm.GEMM_BF16, 128, 16384, 16384, "+splitK(4)(rotated)"), (gemm.GEMM_BF16, 128, 8192, 16384, "+splitK(8)(rotated)"),
                                (gemm.GEMM_F16, 97, 12288, 8192, "+splitK(4)(rotated)"), (gemm.GEMM_F16, 97, 12287, 8192, "+splitK(4)"),
                                (gemm.GEMM_BF16, 128, 8192, 8192, "+splitK(8)"), (gemm.GEMM_BF16, 128, 2048, 4096, "+splitK(4)"),
                                (gemm.GEMM_BF16, 129, 8192, 16384, "+splitK(4)"),
                                (gemm.GEMM_FP8_E4M3, 128, 12288, 16384, "+splitK(4)(rotated)"), (gemm.GEMM_FP8_E4M3, 128, 8192, 16384, "+splitK(8)")]:
        q = gemm.gemm_query(gemm.GEMM_K4_MFMA, gemm.make_desc(M, N, K, dt, gemm.GEMM_F32, ROW, COL, workspace=4096, workspace_bytes=1 << 40))
        assert q.status == gemm.GEMM_OK and q.path == "mfma32-direct-to-lds" + path, (dt, M, N, K, q.path)


def test_how_many_k_ranges_a_streamed_operand_is_read_in():
    """Ranges of whole slabs, as many as fit one round of the 256 CUs; more of them in more rounds where one round leaves so many CUs
    idle that it takes longer; never more than the factor that scratch is asked for.  (A count that divides the factor instead
    leaves one range where the factor is prime.)"""
    bf16, e4m3 = gemm.GEMM_BF16, gemm.GEMM_FP8_E4M3
    for (dt, N, K, ranges) in [(bf16, 16384, 16384, 2), (bf16, 8192, 16384, 4), (bf16, 28672, 4096, 1), (bf16, 20480, 8192, 1), (bf16, 16512, 8192, 1),
                               (bf16, 16384, 10240, 2), (bf16, 16384, 6400, 2), (bf16, 12800, 12800, 2), (bf16, 12288, 20480, 2), (e4m3, 16384, 20480, 2),
                               (bf16, 5120, 20480, 5), (bf16, 5120, 27648, 6), (bf16, 8192, 13888, 7), (bf16, 12800, 8000, 5), (bf16, 8704, 15232, 7),
                               (bf16, 16640, 7104, 3), (bf16, 17408, 12288, 3), (bf16, 20480, 7104, 3), (bf16, 22016, 7104, 1),
                               (bf16, 6400, 17472, 3), (bf16, 10240, 15232, 2), (bf16, 9472, 13888, 7), (bf16, 14336, 9920, 5), (bf16, 7680, 16000, 5)]:
        q = gemm.gemm_query(gemm.GEMM_K4_MFMA, gemm.make_desc(128, N, K, dt, gemm.GEMM_F32, ROW, COL, workspace=4096, workspace_bytes=1 << 40))
        assert q.status == gemm.GEMM_OK and "(rotated)" in q.path and (q.threads, q.bm, q.bn) == (512, 128, 128), q
        assert q.grid == ranges * (N // 128), (N, K, ranges, q)
        assert q.workspace_bytes == int(q.path.split("splitK(")[1][0]) * 128 * N * 4 >= ranges * 128 * N * 4


def _direct_form(M, N, K, dt, la, lb, A=4096, B=4096, **kw):
    out = gemm.GEMM_BF16 if dt == gemm.GEMM_FP8_E4M3 else dt
    q = gemm.gemm_query(gemm.GEMM_K4_MFMA, gemm.make_desc(M, N, K, dt, out, la, lb, **kw), A, B)
    assert q.status == gemm.GEMM_OK and "masked" in q.path, q.path
    return q.path.endswith("(direct-to-lds)")


@pytest.mark.parametrize("dt", [gemm.GEMM_F32, gemm.GEMM_BF16, gemm.GEMM_F16])
def test_addressing_limits_of_the_masked_states_direct_to_lds_form(dt):
    """Rows of 4 MiB where K is contiguous, 2 GiB of k lines (with two slabs of overshoot) where it is not: both sides
    of each limit, for either operand."""
    es = ES[dt]
    row = (1 << 22) // es
    assert _direct_form(70, 65, 33, dt, ROW, ROW, lda=row, ldb=65) and not _direct_form(70, 65, 33, dt, ROW, ROW, lda=row + 1, ldb=65)
    assert _direct_form(70, 65, 33, dt, COL, COL, lda=71, ldb=row) and not _direct_form(70, 65, 33, dt, COL, COL, lda=71, ldb=row + 1)
    for K in (1, 70, 1000):
        line = ((1 << 31) - 1) // es // (K + 2 * 128 // es)
        assert _direct_form(70, 65, K, dt, COL, COL, lda=line, ldb=K + 1) and not _direct_form(70, 65, K, dt, COL, COL, lda=line + 1, ldb=K + 1)
        assert _direct_form(70, 65, K, dt, ROW, ROW, lda=K + 1, ldb=line) and not _direct_form(70, 65, K, dt, ROW, ROW, lda=K + 1, ldb=line + 1)
    assert not _direct_form(70, 65, 33, gemm.GEMM_FP8_E4M3, ROW, ROW)


@pytest.mark.parametrize("dt", [gemm.GEMM_F32, gemm.GEMM_BF16, gemm.GEMM_F16])
@pytest.mark.parametrize("la", [ROW, COL])
@pytest.mark.parametrize("lb", [ROW, COL])
@pytest.mark.parametrize("batch", [1, 3])
def test_an_odd_last_row_at_the_end_of_a_page_keeps_the_element_by_element_kernel(dt, la, lb, batch):
    """Two-byte rows are loaded as dwords from their first element, so an odd-length last row reaches one element past
    the operand: refused where that may not be mapped, whatever the layout and whichever operand."""
    es = ES[dt]
    for odd in (0, 1):
        M, N, K = 130 + odd, 70 + odd, 40 + odd
        ra, ea, rb, eb = (M, K, K, N) if (la, lb) == (ROW, ROW) else (M, K, N, K) if (la, lb) == (ROW, COL) else (K, M, K, N) if lb == ROW else (K, M, N, K)
        kw = dict(lda=ea + 2, ldb=eb + 2, batch=batch, stride_a=ra * (ea + 2), stride_b=rb * (eb + 2))
        end = lambda rows, ext: ((batch - 1) * rows * (ext + 2) + (rows - 1) * (ext + 2) + ext) * es
        at = lambda rows, ext, off: (1 << 20) - end(rows, ext) + off
        for A, B, tail in [(at(ra, ea, 0), 4096, True), (4096, at(rb, eb, 0), True), (at(ra, ea, -es), 4096, False), (4096, at(rb, eb, 4), False)]:
            assert _direct_form(M, N, K, dt, la, lb, A, B, **kw) == (not (tail and odd and es == 2)), (A, B, odd)
