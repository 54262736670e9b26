"""Top-k's short ways on the GPU: one wave that finishes a digit's few keys, and long rows cut into parts, against the oracle or
numpy's stable sort, at the sizes and values where they hand over to the general form."""
import numpy as np
import pytest
import torch

from paper_2605_28213_amd import gemm, topk
from tests.test_topk_gpu import check, run_state

pytestmark = pytest.mark.gpu


def rows(kind, batch, n, ld, rng):
    x = rng.standard_normal((batch, ld)).astype(np.float32)
    if kind == "steps":                       # many elements equal the threshold
        x = np.round(x * 2) / 2
    elif kind == "zeros":                     # one value, of both signs
        x = np.where(x > 0, np.float32(0.0), np.float32(-0.0))
    elif kind == "ascending":                 # the large values are neighbours
        x[:, :n] = np.sort(x[:, :n], axis=1)
    elif kind == "close":                     # keys that differ in their last bits only
        x = (np.float32(1.0) + rng.integers(0, 600, x.shape) * np.float32(2.0 ** -23)).astype(np.float32)
    elif kind == "infinite":
        x[:, ::3] = -np.inf
        x[:, 5::1009] = np.inf
    elif kind == "lowest":
        x[:] = np.finfo(np.float32).min
        x[:, 3::97] = rng.standard_normal(x[:, 3::97].shape)
    x[:, n:] = 1e30
    return x


KINDS = ["normal", "steps", "zeros", "ascending", "close", "infinite", "lowest"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,k", [(5, 2), (600, 511), (3001, 1), (4096, 2048), (4099, 700), (9001, 4000)])
def test_resident_rows(kind, n, k):
    """At most and more than 512 keys in the first digit, rows that leave lanes without elements, four and sixteen keys a lane."""
    check(2, rows(kind, 2, n, (n + 3) // 4 * 4, np.random.default_rng(n + k)), n, k)


def by_sort(x, n, k):
    order = np.argsort(-(x[:, :n].astype(np.float64) + 0.0), axis=1, kind="stable")[:, :k]
    return np.sort(order, axis=1)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("batch,n,ld,k", [(1, 16385, 16385, 1), (3, 16640, 16641, 256), (32, 20481, 20484, 33), (2, 65537, 65537, 100), (2, 49153, 49153, 257), (1, 262144, 262144, 60)])
def test_rows_cut_into_parts(kind, batch, n, ld, k):
    """One element more than whole parts, rows that start at any element, the most rows and the most parts, k up to what the
    second kernel ranks directly and one more, lists that overflow and large values that fall into one part.  Twice: the second
    call finds the slots as the first one left them."""
    x = rows(kind, batch, n, ld, np.random.default_rng(n + k))
    want = by_sort(x, n, k)
    for _ in range(2):
        rc, idx, val, q = run_state(1, x, n, k)
        assert rc == gemm.GEMM_OK and "parts" in q.path and q.grid == batch * -(-n // 4096), q
        np.testing.assert_array_equal(idx, want)
        np.testing.assert_array_equal(val.view(np.uint32), np.take_along_axis(x, want, 1).view(np.uint32))


@pytest.mark.parametrize("kind", KINDS + ["uniform", "shifted", "descending", "sparse"])
@pytest.mark.parametrize("batch,n,k", [(2, 20481, 250), (3, 100001, 60), (2, 100001, 500), (1, 131072, 1500), (2, 262111, 58)])
def test_rows_whose_parts_overflow(kind, batch, n, k):
    """Rows of which the parts cannot list all elements near their bounds: values that share their first digits, equal ones (also
    where only some of a row's are taken), neighbours; k below and above what each part lists."""
    rng = np.random.default_rng(n + k)
    if kind == "uniform":
        x = rng.random((batch, n), dtype=np.float32)
    elif kind == "shifted":
        x = (rng.standard_normal((batch, n)) - 10).astype(np.float32)
    elif kind == "descending":
        x = -np.sort(-rng.standard_normal((batch, n)).astype(np.float32), axis=1)
    elif kind == "sparse":                    # fewer than k above a run of equal values
        x = np.maximum(rng.standard_normal((batch, n)).astype(np.float32) - np.float32(3.5), np.float32(0))
    else:
        x = rows(kind, batch, n, n, rng)
    want = by_sort(x, n, k)
    rc, idx, val, q = run_state(1, x, n, k)
    assert rc == gemm.GEMM_OK and "parts" in q.path, q
    np.testing.assert_array_equal(idx, want)
    np.testing.assert_array_equal(val.view(np.uint32), np.take_along_axis(x, want, 1).view(np.uint32))


@pytest.mark.parametrize("nan", [0x7FFFFFFF, 0xFFFFFFFF, 0x7FC00000, 0xFF800001])
@pytest.mark.parametrize("n,k", [(16385, 256), (20481, 300), (100001, 500)])
def test_rows_with_nans_stay_inside_their_buffers(nan, n, k):
    """The selection of such rows is not defined, but every index written is one of the row's and nothing beside the results is."""
    rng = np.random.default_rng(n)
    bits = rng.standard_normal((3, n)).astype(np.float32).view(np.uint32)
    bits[0, ::7] = nan
    bits[1] = nan
    bits[2, 5:5 + k] = nan
    x = torch.from_numpy(bits.view(np.float32)).cuda()
    idx = torch.full((3 * k + 64,), -7, dtype=torch.int32, device="cuda")
    val = torch.full((3 * k + 64,), -7.0, device="cuda")
    assert topk.topk_run(1, topk.make_desc(3, n, k), x, idx[32:], val[32:]) == gemm.GEMM_OK
    torch.cuda.synchronize()
    for t in (idx, val):
        assert bool((t[:32] == -7).all()) and bool((t[-32:] == -7).all())
    inside = idx[32:-32]
    assert bool(((inside == -7) | ((inside >= 0) & (inside < n))).all())


def test_parts_of_more_rows_than_slots_on_several_streams_and_under_a_graph():
    """Eight streams with 32 rows each in flight at once: rows whose slot another call holds are read uncut, and every result
    is the same; so is that of a graph, replayed among them."""
    n, k, batch = 40000, 50, 32
    gen = torch.Generator(device="cuda").manual_seed(1)
    xs = [torch.randn((batch, n), generator=gen, device="cuda") for _ in range(8)]
    streams = [torch.cuda.Stream() for _ in xs]
    outs = [(torch.zeros((batch, k), dtype=torch.int32, device="cuda"), torch.zeros((batch, k), device="cuda")) for _ in xs]
    want = [torch.sort(torch.sort(x.cpu(), dim=1, descending=True, stable=True).indices[:, :k], dim=1).values for x in xs]
    calls = [(topk.make_desc(batch, n, k, stream=s), x, *o) for s, x, o in zip(streams, xs, outs)]
    graph = torch.cuda.CUDAGraph()
    assert topk.topk_run(1, *calls[0]) == gemm.GEMM_OK
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=streams[0]):
        assert topk.topk_run(1, *calls[0]) == gemm.GEMM_OK
    for _ in range(6):
        for idx, val in outs:
            idx.zero_()
            val.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[0]):
            graph.replay()
        for c in calls[1:]:
            assert topk.topk_run(1, *c) == gemm.GEMM_OK
        torch.cuda.synchronize()
        for x, (idx, val), w in zip(xs, outs, want):
            assert torch.equal(idx.cpu().long(), w) and torch.equal(val, torch.gather(x, 1, idx.long()))
