"""GPU parity of the several-tables-per-launch calls: every table of a batch against the CPU oracle,
and against the single-table calls bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_08679_amd as P
from paper_2010_08679_amd import synth
from util_parity import compare_quantized, u32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BITS = (2, 3, 4, 8)


@pytest.fixture(scope="module")
def ctx():
    c = P.cnr_create(0)
    yield c
    torch.cuda.synchronize()
    P.cnr_destroy(c)


def _poll_clean(ctx):
    assert P.cnr_poll_errors(ctx) == (P.CNR_OK, 0, 0)


class _Tables:
    """A few tables of one row length with ragged sizes, their look-up streams, and both per-table
    and batched checkpointers on the same kind of buffers."""

    def __init__(self, ctx, sizes, dim, seed, n_idx, with_scratch=True, idx_dtype=torch.int64):
        g = torch.Generator(device=DEV).manual_seed(seed)
        self.sizes, self.dim = sizes, dim
        self.tables = [synth.table_outlier_mix(n, dim, 0.02, seed * 100 + i, DEV) for i, n in enumerate(sizes)]
        self.host = [t.cpu().numpy() for t in self.tables]
        self.idx = [None if m == 0 else torch.randint(0, n, (m,), generator=g, device=DEV).to(idx_dtype)
                    for n, m in zip(sizes, n_idx)]

        def cks():
            return [P.TableCheckpointer(ctx, n, dim, device=DEV,
                                        mark_scratch=P.TableCheckpointer.new_mark_scratch(n, DEV) if with_scratch else None)
                    for n in sizes]
        self.single, self.batched = cks(), cks()
        self.batch = P.BatchCheckpointer(ctx, self.batched)

    def oracle_track(self, i):
        bm = O.new_bitmap(self.sizes[i])
        if self.idx[i] is not None:
            O.mark_touched(bm, self.sizes[i], self.idx[i].cpu().numpy())
        ids, n = O.compact_dirty(bm, self.sizes[i])
        return bm, ids, n


def _outputs(cks, bits):
    return [c.alloc_output(bits, want_range=True) for c in cks]


def _host(enc, n, dim, bits):
    prb = P.cnr_packed_row_bytes(dim, bits)
    packed = enc.packed.cpu().numpy()[:n * prb].reshape(n, prb)
    return dict(scale=enc.scale.cpu().numpy()[:n], bias=enc.bias.cpu().numpy()[:n],
                row_min=enc.row_min.cpu().numpy()[:n], row_max=enc.row_max.cpu().numpy()[:n],
                packed=packed, codes=O.unpack(packed, dim, bits))


# small tables share one encode / restore launch, a table of more than 64 MB takes its own
SIZES = {"small": ([70_001, 5_000, 33, 16_384, 1], [300_000, 2_000, 0, 9_000, 3]),   # look-ups: bulk, atomic, none, ...
         "mixed": ([5_000, 300_007, 40_000, 140_000], [4_000, 200_000, 30_000, 90_000])}


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("dim,which", [(64, "small"), (128, "small"), (64, "mixed"), (256, "mixed"), (32, "small")])
def test_batched_checkpoint_equals_oracle_and_single_calls(ctx, bits, dim, which):
    sizes, n_idx = SIZES[which]
    print("case batch %s dim=%d bits=%d" % (which, dim, bits), flush=True)
    T = _Tables(ctx, sizes, dim, seed=bits * 10 + dim, n_idx=n_idx)
    # --- batched path
    T.batch.clear()
    T.batch.mark(T.idx)
    T.batch.compact()
    outs_b = _outputs(T.batched, bits)
    T.batch.encode(T.tables, outs_b)
    stale_b = [torch.zeros_like(t) for t in T.tables]
    T.batch.restore(stale_b, outs_b)
    # --- the same through the single-table calls
    outs_s = _outputs(T.single, bits)
    stale_s = [torch.zeros_like(t) for t in T.tables]
    for c, idx, t, o, st in zip(T.single, T.idx, T.tables, outs_s, stale_s):
        c.clear()
        if idx is not None:
            c.mark(idx)
        c.compact()
        c.encode(t, o)
        c.restore(st, o)
    torch.cuda.synchronize()
    for i, n_rows in enumerate(sizes):
        bm, ids, n = T.oracle_track(i)
        cb, cs = T.batched[i], T.single[i]
        assert np.array_equal(u32(cb.bitmap)[:bm.size], bm), "table %d bitmap" % i
        assert int(cb.n_dirty.item()) == n and np.array_equal(u32(cb.row_ids)[:n], ids)
        if cb.mark_scratch is not None:
            assert not cb.mark_scratch.any()
        got = _host(outs_b[i], n, dim, bits)
        one = _host(outs_s[i], n, dim, bits)
        for k in ("scale", "bias", "row_min", "row_max", "packed"):
            assert np.array_equal(got[k], one[k]), "table %d %s differs from the single-table call" % (i, k)
        assert torch.equal(stale_b[i], stale_s[i])
        if n:
            ora = O.quantize_rows(T.host[i], ids, bits, n_threads=8)
            compare_quantized(T.host[i][ids], got, ora, bits, what="batch table %d b%d d%d" % (i, bits, dim))
            want = np.zeros_like(T.host[i])
            O.restore_rows(want, ids, bits, got["packed"], got["scale"], got["bias"])
            assert np.array_equal(stale_b[i].cpu().numpy(), want)
    _poll_clean(ctx)


@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
def test_batched_mark_takes_each_table_by_its_own_route(ctx, dtype):
    # one batch whose tables need all three routes of the mark: bitmap slices in LDS with teams of one,
    # two and three workgroups (four tables with long streams, so that the call's estimate favours the
    # slices for them), flag bytes for a table too large for that, atomics for short streams
    slice_rows = 32 * 40960
    sizes = [3 * slice_rows - 5, 100, 16 * slice_rows + 77, slice_rows + 1, 40_000, slice_rows, 2 * slice_rows + 3, slice_rows - 1]
    n_idx = [400_001, 50, 500_003, 300_000, 100, 0, 390_000, 380_003]
    print("case mixed-route mark dtype=%s" % dtype, flush=True)
    g = torch.Generator(device=DEV).manual_seed(77)
    cks = [P.TableCheckpointer(ctx, n, 16, device=DEV, mark_scratch=P.TableCheckpointer.new_mark_scratch(n, DEV))
           for n in sizes]
    batch = P.BatchCheckpointer(ctx, cks)
    idx = [None if m == 0 else torch.randint(-1, n + 1, (m,), generator=g, device=DEV).to(dtype)
           for n, m in zip(sizes, n_idx)]
    batch.clear()
    batch.mark(idx)
    batch.mark(idx)                                            # marks accumulate; the same streams again
    batch.compact()
    torch.cuda.synchronize()
    skipped = 0
    for i, n_rows in enumerate(sizes):
        bm = O.new_bitmap(n_rows)
        if idx[i] is not None:
            skipped += 2 * O.mark_touched(bm, n_rows, idx[i].cpu().numpy())
        ids, n = O.compact_dirty(bm, n_rows)
        assert np.array_equal(u32(cks[i].bitmap)[:bm.size], bm), "table %d bitmap" % i
        assert int(cks[i].n_dirty.item()) == n and np.array_equal(u32(cks[i].row_ids)[:n], ids)
        assert not cks[i].mark_scratch.any()
    st, bad, flags = P.cnr_poll_errors(ctx)
    assert st == P.CNR_E_INDEX_RANGE and bad == skipped and skipped > 0 and flags == 0
    _poll_clean(ctx)


@pytest.mark.parametrize("bits,dim", [(4, 64), (2, 128), (3, 256)])
def test_batched_greedy(ctx, bits, dim):
    sizes = [3_001, 700, 64]
    T = _Tables(ctx, sizes, dim, seed=7 + bits, n_idx=[2_500, 900, 64])
    T.batch.clear()
    T.batch.mark(T.idx)
    T.batch.compact()
    outs = _outputs(T.batched, bits)
    T.batch.encode(T.tables, outs, mode=P.CNR_RANGE_GREEDY, greedy=(20, 0.6))
    torch.cuda.synchronize()
    for i in range(len(sizes)):
        _, ids, n = T.oracle_track(i)
        got = _host(outs[i], n, dim, bits)
        ora = O.quantize_rows(T.host[i], ids, bits, mode=O.RANGE_GREEDY, num_bins=20, ratio=0.6, n_threads=8)
        compare_quantized(T.host[i][ids], got, ora, bits, greedy=True, what="batch greedy table %d" % i)
    _poll_clean(ctx)


def test_more_tables_than_one_launch_takes(ctx):
    n_tables = P.CNR_MAX_BATCH + 3
    sizes = [1_000 + 37 * i for i in range(n_tables)]
    T = _Tables(ctx, sizes, 64, seed=3, n_idx=[400 + i for i in range(n_tables)], with_scratch=False,
                idx_dtype=torch.int32)
    T.batch.clear()
    T.batch.mark(T.idx)
    T.batch.compact()
    outs = _outputs(T.batched, 4)
    T.batch.encode(T.tables, outs)
    stale = [torch.zeros_like(t) for t in T.tables]
    T.batch.restore(stale, outs)
    torch.cuda.synchronize()
    for i in range(n_tables):
        bm, ids, n = T.oracle_track(i)
        assert np.array_equal(u32(T.batched[i].bitmap)[:bm.size], bm)
        assert int(T.batched[i].n_dirty.item()) == n and np.array_equal(u32(T.batched[i].row_ids)[:n], ids)
        got = _host(outs[i], n, 64, 4)
        ora = O.quantize_rows(T.host[i], ids, 4)
        compare_quantized(T.host[i][ids], got, ora, 4, what="table %d of %d" % (i, n_tables))
        want = np.zeros_like(T.host[i])
        O.restore_rows(want, ids, 4, got["packed"], got["scale"], got["bias"])
        assert np.array_equal(stale[i].cpu().numpy(), want)
    _poll_clean(ctx)


def test_other_row_lengths_go_table_by_table(ctx):
    sizes = [900, 2_000]
    T = _Tables(ctx, sizes, 40, seed=11, n_idx=[500, 1_500])
    T.batch.clear()
    T.batch.mark(T.idx)
    T.batch.compact()
    outs = _outputs(T.batched, 4)
    T.batch.encode(T.tables, outs)
    stale = [torch.zeros_like(t) for t in T.tables]
    T.batch.restore(stale, outs)
    torch.cuda.synchronize()
    for i in range(2):
        _, ids, n = T.oracle_track(i)
        got = _host(outs[i], n, 40, 4)
        ora = O.quantize_rows(T.host[i], ids, 4)
        compare_quantized(T.host[i][ids], got, ora, 4, what="dim 40 table %d" % i)
        want = np.zeros_like(T.host[i])
        O.restore_rows(want, ids, 4, got["packed"], got["scale"], got["bias"])
        assert np.array_equal(stale[i].cpu().numpy(), want)
    _poll_clean(ctx)


def test_bad_job_rejects_the_whole_call_before_any_launch(ctx):
    T = _Tables(ctx, [2_000, 2_000], 64, seed=5, n_idx=[1_000, 1_000])
    T.batch.clear()
    torch.cuda.synchronize()
    jobs = T.batch.jobs(indices=T.idx)
    jobs[1].n_rows = 1 << 32
    with pytest.raises(P.CnrError) as e:
        P.cnr_mark_touched_batch(ctx, jobs, P.CNR_IDX_I64)
    assert e.value.status == P.CNR_E_INVALID
    jobs = T.batch.jobs(indices=T.idx)
    jobs[1].indices += 4                                       # int64 stream at a 4-byte boundary
    with pytest.raises(P.CnrError) as e:
        P.cnr_mark_touched_batch(ctx, jobs, P.CNR_IDX_I64)
    assert e.value.status == P.CNR_E_ALIGN
    torch.cuda.synchronize()
    assert not T.batched[0].bitmap.any() and not T.batched[1].bitmap.any()
    outs = _outputs(T.batched, 4)
    with pytest.raises(P.CnrError) as e:
        P.cnr_quantize_rows_batch(ctx, T.batch.jobs(tables=T.tables, outs=outs), 64, 5, P.CNR_RANGE_MINMAX)
    assert e.value.status == P.CNR_E_BITS
    with pytest.raises(P.CnrError) as e:
        P.cnr_restore_rows_batch(ctx, T.batch.jobs(tables=T.tables, outs=outs), 12, 3)
    assert e.value.status == P.CNR_E_DIM
    _poll_clean(ctx)


def test_capacity_overflow_in_one_table_of_a_batch(ctx):
    sizes = [4_000, 4_000]
    cks = [P.TableCheckpointer(ctx, sizes[0], 64, device=DEV),
           P.TableCheckpointer(ctx, sizes[1], 64, capacity=100, device=DEV)]
    batch = P.BatchCheckpointer(ctx, cks)
    g = torch.Generator(device=DEV).manual_seed(9)
    idx = [torch.randint(0, n, (3_000,), generator=g, device=DEV) for n in sizes]
    batch.clear()
    batch.mark(idx)
    cks[1].row_ids.fill_(-1)
    batch.compact()
    st, bad, flags = P.cnr_poll_errors(ctx)
    assert st == P.CNR_E_CAPACITY and flags == P.CNR_FLAG_CAPACITY and bad == 0
    for c, ix in zip(cks, idx):
        bm = O.new_bitmap(c.n_rows)
        O.mark_touched(bm, c.n_rows, ix.cpu().numpy())
        ids, n = O.compact_dirty(bm, c.n_rows)
        assert int(c.n_dirty.item()) == n                      # the true count, also when truncated
        m = min(n, c.capacity)
        assert np.array_equal(u32(c.row_ids)[:m], ids[:m])
    _poll_clean(ctx)


def test_batched_step_replays_from_a_hip_graph(ctx):
    # the batched calls only enqueue kernels on the caller's stream (job descriptors travel by value in
    # the launch), so a whole step over several tables can be captured once and replayed; inputs are
    # refreshed in place between replays and every replay is checked against the oracle
    sizes, dim, bits = [90_001, 20_000, 50], 64, 4
    T = _Tables(ctx, sizes, dim, seed=21, n_idx=[200_000, 5_000, 40])
    outs = _outputs(T.batched, bits)
    stale = [torch.zeros_like(t) for t in T.tables]

    def step():                                                 # prepared calls hold the stream that is
        for _, call in T.batch.prepare_step(T.idx, T.tables, outs, restore_into=stale):  # current here
            call()

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                                  # warm-up outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    g = torch.Generator(device=DEV).manual_seed(77)
    for rep in range(3):
        for i, n_rows in enumerate(sizes):                      # eager work between the replays
            T.idx[i].copy_(torch.randint(0, n_rows, (T.idx[i].numel(),), generator=g, device=DEV))
            T.tables[i].mul_(1.0 + 0.1 * (rep + 1))
            stale[i].fill_(float(rep))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, n_rows in enumerate(sizes):
            host = T.tables[i].cpu().numpy()
            _, ids, n = T.oracle_track(i)
            c = T.batched[i]
            assert int(c.n_dirty.item()) == n and np.array_equal(u32(c.row_ids)[:n], ids)
            got = _host(outs[i], n, dim, bits)
            ora = O.quantize_rows(host, ids, bits, n_threads=8)
            compare_quantized(host[ids], got, ora, bits, what="replay %d table %d" % (rep, i))
            want = np.full_like(host, float(rep))
            O.restore_rows(want, ids, bits, got["packed"], got["scale"], got["bias"])
            assert np.array_equal(stale[i].cpu().numpy(), want)
            assert not c.mark_scratch.any()
    _poll_clean(ctx)


class _Sub(torch.Tensor):
    pass


def test_packed_jobs_are_the_general_ones(ctx):
    """The extension's addresses and refusals against the general checks, also for parameters and subclasses."""
    import ctypes

    f, i, l, u = (torch.zeros(8, dtype=d, device=DEV) for d in (torch.float32, torch.int32, torch.int64, torch.uint8))
    jobs = [dict(table=torch.nn.Parameter(f), n_rows=3, bitmap=i, indices=l, mark_scratch=u, row_ids=i[4:], capacity=5, n_dirty_dev=l[1:],
                 compact_scratch=l, scale=f, bias=f.as_subclass(_Sub), row_min=None, row_max=f[:0], codes_u8=u, packed=u[1:]),
            dict(n_rows=2 ** 32 - 1, table=f)]
    want = bytes(P.binding.make_jobs(jobs))
    fields = [n for n, _ in P.binding.cnr_table_job._fields_]
    rows = [tuple(j.get(k, j["indices"].numel() if k == "n_indices" and "indices" in j else 0) for k in fields) for j in jobs]
    assert P.binding.job_bytes(rows) == want and len(want) == 2 * ctypes.sizeof(P.binding.cnr_table_job)
    assert P.binding.job_bytes([]) == b""
    for t, dtype in ((f, torch.int32), (f[::2], None), (f.as_subclass(_Sub)[::2], None), (f.cpu(), None), (f.cpu().as_subclass(_Sub), None),
                     (7.5, None), ([f], None)):
        raised = []
        for check in (P.binding._dev, P.binding._general_dev):
            with pytest.raises((TypeError, ValueError)) as e:
                check(t, dtype, "table")
            raised.append((e.type, str(e.value)))
        assert raised[0] == raised[1]
    for bad in ([(0,) * 15], [[0] * 16], [(i,) + (0,) * 15], [(0, -1) + (0,) * 14]):
        with pytest.raises((TypeError, OverflowError)):
            P.binding.job_bytes(bad)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert P.binding._stream(None) == s.cuda_stream == P.binding._stream(s)
    assert P.binding._stream(None) == torch.cuda.current_stream().cuda_stream


def test_a_tensor_that_throws_leaves_no_job_behind(ctx):
    import sys

    def inside(t):   # a tensor without memory of its own: its address is refused by an exception, not by a check
        row = (t, 1) + (0,) * 14
        before = sys.getrefcount(t), sys.getrefcount(row)
        for _ in range(3):
            with pytest.raises(RuntimeError):
                P.binding.job_bytes([row])
        assert (sys.getrefcount(t), sys.getrefcount(row)) == before
        return t

    torch.vmap(inside)(torch.zeros(2, 8, device=DEV))


# other row lengths: more tables than a launch takes, lists on either side of a row per wave (448: 32,768 rows), large tables
# (rows of over 64 MB) between small ones, an empty one, counts on the device and lengths the host knows, bad row ids
@pytest.mark.parametrize("dim,bits,sizes", [
    (8, 3, [1, 3000, 0, 2_200_000, 77, 98_400, 16, 5] + [40] * 11), (96, 4, [200_000, 3, 12_300, 999]), (100, 2, [17, 5000, 6200]),
    (448, 8, [32_768, 32_769, 40, 45_000, 33_000]), (600, 4, [70, 30_000, 1])])
def test_other_row_lengths_share_launches(ctx, dim, bits, sizes):
    print("case shared launches dim=%d bits=%d" % (dim, bits), flush=True)
    g = torch.Generator(device=DEV).manual_seed(dim)
    prb = P.cnr_packed_row_bytes(dim, bits)
    jobs, single, keep = [], [], []
    for i, n in enumerate(sizes):
        cap = max(1, n)
        rows = cap + 7
        table = torch.randn(rows, dim, device=DEV, generator=g) * 0.05
        ids = torch.sort(torch.randperm(rows, device=DEV, generator=g)[:cap]).values.to(torch.int32)
        if n > 20 and i % 2:
            ids[[0, n // 2, n - 1]] = rows + 3
        live = torch.tensor([n - n // 3], dtype=torch.int64, device=DEV) if i % 3 else None
        out = [[torch.full((cap * w,), fill, dtype=d, device=DEV) for d, w, fill in
                ((torch.float32, 1, -7.0), (torch.float32, 1, -7.0), (torch.float32, 1, -7.0), (torch.uint8, prb, 0xEE), (torch.float32, 0, 0.0))]
               for _ in range(2)]
        back = [torch.zeros_like(table) for _ in range(2)]
        s, b, mn, pk, _ = out[0]
        jobs.append(dict(table=table, n_rows=rows, row_ids=ids, capacity=n, n_dirty_dev=live, scale=s, bias=b, row_min=mn, packed=pk))
        single.append((table, rows, ids, live, n, out[1]))
        keep.append((out, back))
    P.cnr_quantize_rows_batch(ctx, jobs, dim, bits, P.CNR_RANGE_MINMAX)
    for j, (_, back) in zip(jobs, keep):
        j["table"] = back[0]
    P.cnr_restore_rows_batch(ctx, jobs, dim, bits)
    for (table, rows, ids, live, n, (s, b, mn, pk, _)), (_, back) in zip(single, keep):
        if n:
            P.cnr_quantize_rows(ctx, table, rows, dim, ids, live, n, bits, P.CNR_RANGE_MINMAX, None, s, b, row_min=mn, packed=pk)
            P.cnr_restore_rows(ctx, back[1], rows, dim, ids, live, n, bits, pk, s, b)
    torch.cuda.synchronize()
    for i, (out, back) in enumerate(keep):
        for k, (x, y) in enumerate(zip(out[0] + [back[0]], out[1] + [back[1]])):
            assert torch.equal(x, y), (i, sizes[i], k)
        assert sizes[i] < 20 or bool(back[0].any())
    st, bad, flags = P.cnr_poll_errors(ctx)
    assert bad == 0 and flags == P.CNR_FLAG_ROW_ID and st != P.CNR_OK


def test_job_arrays_from_the_extension_are_those_of_the_general_way(ctx, monkeypatch):
    # what the extension packs in one step against field by field, and what it leaves to that: everything out of the ordinary
    from paper_2010_08679_amd import binding as B
    sent = []
    for name in ("cnr_clear_bitmap_batch", "cnr_mark_touched_batch", "cnr_compact_dirty_batch", "cnr_quantize_rows_batch", "cnr_restore_rows_batch"):
        monkeypatch.setattr(B, name, lambda ctx, jobs, *rest, name=name: sent.append((name, bytes(jobs), rest)))
    n_rows, dim = (50, 1_000, 33), 24
    cks = [P.TableCheckpointer(ctx, n, dim, capacity=c, device=DEV, mark_scratch=P.TableCheckpointer.new_mark_scratch(n, DEV) if n != 33 else None)
           for n, c in zip(n_rows, (50, 7, 0))]
    batch = P.BatchCheckpointer(ctx, cks)
    tables = [torch.zeros(n, dim, device=DEV) for n in n_rows]
    fast, took = B.batch_jobs, []

    def counting(*args):
        took.append(fast(*args))
        return took[-1]

    def both(call, by_extension):
        def outcome(f):
            monkeypatch.setattr(B, "batch_jobs", f)
            sent.clear()
            try:
                call()
            except Exception as e:
                return type(e)
            return list(sent)
        took.clear()
        one, other = outcome(counting), outcome(lambda *a: None)
        assert one == other and len(took) == 1 and (took[0] is not None) == by_extension, (one, other, took)

    both(batch.clear, True)
    both(batch.compact, True)
    ix = [torch.arange(5, device=DEV), None, torch.arange(6, device=DEV).reshape(2, 3)]
    both(lambda: batch.mark(ix), True)
    both(lambda: batch.mark(tuple(t if t is None else t.int() for t in ix) + (None,)), True)
    for odd in (ix[:2], [None] * 3, [ix[0], ix[0].int(), None], [torch.arange(9, device=DEV)[::2], None, None], [ix[0].cpu(), None, None], [ix[0].short(), None, None],
                [3, None, None], dict(enumerate(ix))):
        both(lambda: batch.mark(odd), False)
    for bits, ranges in ((2, False), (3, True), (4, True), (8, False)):
        outs = [c.alloc_output(bits, want_range=ranges) for c in cks]
        both(lambda: batch.encode(tables, outs), True)
        both(lambda: batch.restore(tuple(tables), outs), True)
        for i, field in ((0, "scale"), (1, "bias"), (2, "packed")):
            good = getattr(outs[i], field)
            for bad in (None, good[:-1], good.cpu(), good.double()):
                setattr(outs[i], field, bad)
                both(lambda: batch.encode(tables, outs), False)
            setattr(outs[i], field, good)
        for bad in (tables[:2], [tables[0], tables[1].t().contiguous().t(), tables[2]], [tables[0], tables[1][:-1], tables[2]], [tables[0].half()] + tables[1:], [None] + tables[1:]):
            both(lambda: batch.restore(bad, outs), False)
    ids, cks[0].row_ids = cks[0].row_ids, cks[0].row_ids.long()
    both(batch.compact, False)
    cks[0].row_ids, cks[1].n_rows = ids, -1
    both(batch.clear, False)
    cks[1].n_rows = True
    both(batch.clear, False)


def test_look_ups_beyond_the_tables_share_the_dtype_too(ctx):
    # tensors beyond the last table are not marked, but a dtype of their own, or no dtype, is refused as it is among the tables' own
    cks = [P.TableCheckpointer(ctx, 100, 16, device=DEV) for _ in range(2)]
    batch = P.BatchCheckpointer(ctx, cks)
    ix = [torch.tensor([3 * i + 1], device=DEV) for i in range(3)]
    for seq in (list, tuple):
        batch.clear()
        for more in ([ix[2]], [None], [ix[2], None, ix[2].cpu()], []):
            batch.mark(seq(ix[:2] + more))
        assert [torch.nonzero(c.bitmap).numel() for c in cks] == [1, 1]
        assert [int(c.bitmap[0]) for c in cks] == [2, 16]
        for more, error in (([ix[2].int()], TypeError), ([None, ix[2].int()], TypeError), ([3], AttributeError)):
            with pytest.raises(error):
                batch.mark(seq(ix[:2] + more))
    assert P.cnr_poll_errors(ctx)[1:] == (0, 0)
