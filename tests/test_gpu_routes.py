"""The dispatch branches of the row kernels at the sizes where they can go wrong: list lengths on either
side of a branch, remainders of lane groups and workgroups, row lengths that are no power of two,
unaligned tables, counts on the device below the capacity, ids outside the table."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_08679_amd as P
from paper_2010_08679_amd import synth
from util_parity import GpuTable, compare_greedy, compare_quantized, gpu_encode_all_outputs, tie_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    c = P.cnr_create(0)
    yield c
    torch.cuda.synchronize()
    P.cnr_destroy(c)


def _poll(ctx, want_flags=0):
    st, bad, flags = P.cnr_poll_errors(ctx)
    assert (bad, flags) == (0, want_flags) and (st == P.CNR_OK) == (want_flags == 0)


def _unpack(packed, n, dim, bits):
    """Codes [n, dim] (float32) of densely packed rows."""
    out = torch.zeros((n, dim), dtype=torch.float32, device=packed.device)
    b = packed[:n * dim * bits // 8].view(n, -1)
    for t in range(bits):
        pos = torch.arange(dim, device=packed.device) * bits + t
        out += ((b[:, pos >> 3] >> (pos & 7).to(torch.uint8)) & 1).float() * float(1 << t)
    return out


def _ids(n_rows, n, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.sort(torch.randperm(n_rows, generator=g, device=DEV)[:n]).values.to(torch.int32)


# ---- error metric: by units or a wave per row, the mean in one step or by workgroups' parts -----------

@pytest.mark.parametrize("dim,bits,n,shift", [
    (64, 4, 1, 0), (64, 3, 63, 0), (64, 2, 16_384, 0), (64, 8, 16_385, 0), (64, 2, 600_001, 0),   # 16 lanes per row; past the grid's cap
    (24, 3, 20_011, 0), (20, 2, 40_003, 0), (40, 3, 16_400, 0),                                  # 8 lanes
    (12, 4, 70_001, 0), (4, 8, 16_641, 0), (4, 2, 300, 0),                                       # 4 lanes
    (100, 2, 17_001, 0), (96, 3, 33_000, 0), (512, 4, 16_500, 0),                                # several trips, the last one partial
    (516, 4, 16_500, 0), (1024, 3, 16_500, 0), (1028, 2, 16_500, 0), (4096, 8, 5_000, 0),        # 32 and 64 lanes
    (64, 4, 20_001, 1), (64, 4, 500, 1), (6, 4, 40_001, 0),                                      # a wave per row: unaligned table, odd dim
])
def test_error_metric_routes(ctx, dim, bits, n, shift):
    print("case error dim=%d bits=%d n=%d shift=%d" % (dim, bits, n, shift), flush=True)
    n_rows = n + n // 3 + 5
    table = synth.table_outlier_mix(n_rows, dim, 0.02, dim + bits, DEV)
    ids = _ids(n_rows, n, n)
    scale = torch.empty(n, dtype=torch.float32, device=DEV)
    bias = torch.empty_like(scale)
    g = torch.Generator(device=DEV).manual_seed(7)
    if dim % 4 == 0:
        packed = torch.empty(n * P.cnr_packed_row_bytes(dim, bits), dtype=torch.uint8, device=DEV)
        P.cnr_quantize_rows(ctx, table, n_rows, dim, ids, None, n, bits, P.CNR_RANGE_MINMAX, None, scale, bias, packed=packed)
    else:  # the encoder takes no such rows; any codes will do
        packed = torch.randint(0, 256, (n * P.cnr_packed_row_bytes(dim, bits),), generator=g, device=DEV, dtype=torch.uint8)
        scale.uniform_(0.001, 0.01, generator=g)
        bias.uniform_(-0.1, 0.0, generator=g)
    if shift:
        moved = torch.empty(n_rows * dim + shift, dtype=torch.float32, device=DEV)[shift:].view(n_rows, dim)
        table = moved.copy_(table)
    back = _unpack(packed, n, dim, bits) * scale[:, None] + bias[:, None]
    want = (table[ids.long()].double() - back.double()).square().sum(1).sqrt()
    # the count on the device: either side of a short list and of one with partial sums
    first = None
    for live in sorted({n, max(1, n - 777), n // 2, 0} | {k for k in (1, 128, 129, 8192, 8193, 16_384, 16_385) if k <= n}):
        n_dev = torch.tensor([live], dtype=torch.int64, device=DEV)
        err = torch.full((n,), -1.0, dtype=torch.float64, device=DEV)
        mean = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
        P.cnr_quant_error(ctx, table, n_rows, dim, ids, n_dev, n, bits, packed, scale, bias, err, mean)
        # fp64 sums of at most 600,001 terms added up in another order: 64 roundings for a row; for the mean
        # a few hundred along any path of the summation tree
        assert torch.allclose(err[:live], want[:live], rtol=1e-14, atol=0) and bool((err[live:] == -1.0).all())
        assert float(mean) == pytest.approx(float(want[:live].mean()) if live else 0.0, rel=1e-13)
        again = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
        P.cnr_quant_error(ctx, table, n_rows, dim, ids, n_dev, n, bits, packed, scale, bias, err, again)
        assert float(again) == float(mean)                     # a fixed order
        plain = torch.full((n,), -1.0, dtype=torch.float64, device=DEV)
        P.cnr_quant_error(ctx, table, n_rows, dim, ids, n_dev, n, bits, packed, scale, bias, plain, None)
        assert torch.equal(plain, err)                         # without a mean: the same errors
        if live >= 128:                                        # and in lists of other lengths
            first = err[:128].clone() if first is None else first
            assert torch.equal(err[:128], first)
    _poll(ctx)


@pytest.mark.parametrize("n", [1000, 20_000])
def test_error_metric_skips_ids_outside_the_table(ctx, n):
    dim, bits, n_rows = 64, 4, 30_000
    table = synth.table_normal(n_rows, dim, 0.05, 3, DEV)
    ids = _ids(n_rows, n, 5)
    scale = torch.full((n,), 0.01, dtype=torch.float32, device=DEV)
    bias = torch.full((n,), -0.1, dtype=torch.float32, device=DEV)
    packed = torch.full((n * 32,), 0x5A, dtype=torch.uint8, device=DEV)
    back = _unpack(packed, n, dim, bits) * scale[:, None] + bias[:, None]
    want = (table[ids.long()].double() - back.double()).square().sum(1).sqrt()
    for k in (0, 64, 65, n - 1):                               # a workgroup's first row among them
        ids[k] = n_rows + k
        want[k] = 0.0
    err = torch.full((n,), -1.0, dtype=torch.float64, device=DEV)
    mean = torch.zeros(1, dtype=torch.float64, device=DEV)
    P.cnr_quant_error(ctx, table, n_rows, dim, ids, None, n, bits, packed, scale, bias, err, mean)
    assert torch.allclose(err, want, rtol=1e-14, atol=0)
    assert float(mean) == pytest.approx(float(want.mean()), rel=1e-13)
    _poll(ctx, P.CNR_FLAG_ROW_ID)


@pytest.mark.parametrize("dim,bits,n", [
    (20, 8, 3_001), (32, 4, 129), (36, 2, 16_385), (40, 3, 130), (60, 4, 9_001), (72, 8, 2_049), (92, 2, 700), (96, 4, 16_400), (100, 8, 300),
    (116, 4, 1_025), (120, 3, 16_390), (128, 2, 128), (132, 4, 2_000), (160, 8, 131), (200, 3, 17_003), (240, 4, 8_200), (256, 3, 8_193),
    (500, 2, 1_000), (512, 8, 140)])
def test_error_metric_lanes(ctx, dim, bits, n):
    test_error_metric_routes(ctx, dim, bits, n, 0)


# lanes per row of the restore: whole lines and shared ones at the lengths where the rule changes
@pytest.mark.parametrize("dim,bits", [(64 - 4, 4), (68, 2), (72, 3), (80, 4), (92, 2), (96, 3), (100, 8), (112, 2), (124, 4), (132, 2), (144, 3), (188, 8),
                                      (192, 4), (196, 2), (208, 3), (252, 8), (260, 4)])
def test_restore_lanes(ctx, dim, bits):
    for n in (1, 5, 3_003):
        n_rows = n + n // 2 + 3
        g = torch.Generator(device=DEV).manual_seed(dim + n)
        ids = _ids(n_rows, n, dim)
        packed = torch.randint(0, 256, (n * P.cnr_packed_row_bytes(dim, bits),), generator=g, device=DEV, dtype=torch.uint8)
        scale = torch.empty(n, device=DEV).uniform_(0.001, 0.01, generator=g)
        bias = torch.empty(n, device=DEV).uniform_(-0.1, 0.0, generator=g)
        want = torch.full((n_rows, dim), 7.0, device=DEV)
        table = want.clone()
        rows = _unpack(packed, n, dim, bits) * scale[:, None] + bias[:, None]
        live = max(1, n - 2)
        want[ids[:live].long()] = rows[:live]
        P.cnr_restore_rows(ctx, table, n_rows, dim, ids, torch.tensor([live], dtype=torch.int64, device=DEV), n, bits, packed, scale, bias)
        assert torch.equal(table, want), n
        P.cnr_restore_rows(ctx, table, n, dim, None, None, n, bits, packed, scale, bias)
        assert torch.equal(table[:n], rows) and torch.equal(table[n:], want[n:]), n
    _poll(ctx)


# ---- greedy search at row lengths that are no power of two: lanes per row, units per lane, list length --

def _special_rows(dim, seed):
    """Rows a few float spacings wide, constant, huge and tiny rows: waves that hold one search by division."""
    rng = np.random.default_rng(seed)
    rows = [np.full((2, dim), 0.25, dtype=np.float32), np.float32(rng.normal(0, 1e30, size=(2, dim))),
            np.float32(rng.normal(0, 1e-36, size=(2, dim)))]
    for base in (np.float32(1.0), np.float32(-7.5)):
        u = np.spacing(np.abs(base))
        for span in (1, 7, 3000):
            x = (base + u * rng.integers(0, span + 1, size=(2, dim)).astype(np.float32)).astype(np.float32)
            x[:, 0], x[:, 1] = base, base + u * span
            rows.append(x)
    return np.concatenate(rows)


@pytest.mark.parametrize("dim,bits,wide", [
    (4, 8, 9_830), (8, 3, 24_576), (24, 3, 49_152), (28, 4, 57_344), (24, 8, 19_660),   # a lane per row / twice four
    (36, 2, 24_576), (40, 3, 24_576), (48, 8, 9_830), (68, 4, 34_816),              # two lanes / twice eight
    (72, 3, 23_040), (96, 3, 26_624), (100, 4, 26_624), (140, 2, 26_624),           # four, eight units at most / twice eight
    (144, 3, 46_080), (268, 2, 85_760),                                             # four, sixteen units / twice eight
    (272, 3, 5_440), (284, 2, 5_680),                                               # twice eight at any length
    (288, 4, 5_760), (320, 8, 2_560), (1084, 2, 21_680),                            # sixteen / twice thirty-two
    (1088, 3, 1_000), (2044, 4, 500), (4096, 2, 300),                               # sixty-four
])
def test_greedy_routes_of_other_row_lengths(ctx, dim, bits, wide):
    print("case greedy units dim=%d bits=%d" % (dim, bits), flush=True)
    n_rows = wide + wide // 8 + 77
    table = synth.table_outlier_mix(n_rows, dim, 0.02, dim + bits, DEV)
    rng = np.random.default_rng(dim)
    special = _special_rows(dim, dim + 1)
    where = np.sort(rng.choice(n_rows, size=special.shape[0], replace=False))
    table[torch.from_numpy(where).to(DEV)] = torch.from_numpy(special).to(DEV)
    gt = GpuTable(ctx, table)
    # to the last iteration, where the candidates are narrowest (8 bits meet exact ties there), and a part of the way
    for params in ({2: (25, 1.0), 3: (25, 1.0), 4: (45, 1.0), 8: (20, 1.0)}[bits], (12, 0.33)):
        for n in (wide + 5, wide - 3, 17):  # on the device alone: the buffers' capacity allows the long form
            with_special = where[:min(n, len(where))]   # exactly n rows: they decide between the forms
            ids = np.sort(np.concatenate([with_special, rng.choice(np.setdiff1d(np.arange(n_rows), with_special), size=n - len(with_special), replace=False)]))
            gt.ck.clear()
            gt.ck.mark(torch.from_numpy(ids).to(DEV))
            gt.ck.compact()
            got = gpu_encode_all_outputs(gt, bits, mode=P.CNR_RANGE_GREEDY, greedy=params)
            assert got["n"] == ids.size
            rows = gt.host[ids]
            assert np.array_equal(got["row_min"], rows.min(axis=1)) and np.array_equal(got["row_max"], rows.max(axis=1))
            assert np.array_equal(got["packed"], O.pack(got["codes"], bits))
            pos = np.unique(np.concatenate([np.arange(min(40, ids.size)), np.arange(max(0, ids.size - 40), ids.size),
                                            np.flatnonzero(np.isin(ids, where)), rng.integers(0, ids.size, size=1500)]))
            ora = O.quantize_rows(rows[pos], None, bits, mode=O.RANGE_GREEDY, num_bins=params[0], ratio=params[1], n_threads=8)
            compare_greedy(rows[pos], {k: got[k][pos] for k in ("scale", "bias", "row_min", "row_max", "codes")}, ora, bits, *params,
                           what="greedy units b%d d%d n%d" % (bits, dim, n))
    _poll(ctx)


@pytest.mark.parametrize("dim,bits,limit", [(16, 4, 24_576), (32, 3, 24_576), (64, 2, 12_288), (64, 3, 12_288), (64, 4, 12_288), (64, 8, 12_288), (128, 3, 12_288),
                                            (256, 4, 6_144), (16, 8, 6_144), (32, 8, 6_144)])
def test_greedy_short_lists_of_power_of_two_rows(ctx, dim, bits, limit):
    # up to `limit` rows (a bound the host knows) two groups of lanes per row, beyond it one; whole searches of rows of 64 at 3 and 4 bits
    # up to two thirds of it, at 8 bits rows of 64 and more not at all
    n_rows = limit + 3
    table = synth.table_outlier_mix(n_rows, dim, 0.02, dim + bits, DEV)
    rng = np.random.default_rng(dim)
    special = _special_rows(dim, dim + 1)
    where = np.sort(rng.choice(n_rows - 5, size=special.shape[0], replace=False))
    table[torch.from_numpy(where).to(DEV)] = torch.from_numpy(special).to(DEV)
    gt = GpuTable(ctx, table)
    # up to its last iteration, and a few and the fewest iterations, whose lines lie lower
    many, few = {2: (25, 1.0), 3: (25, 1.0), 4: (45, 1.0), 8: (20, 1.0)}[bits], (12, 0.75)
    lines = [(many, limit * 2 // 3 if dim == 64 and bits in (3, 4) else limit), (few, limit // 2 if dim <= 64 else limit // 4), ((12, 0.1), limit // 4),
             ((100, 0.17), limit)]
    for params, line in lines:
        for n in (1, 77, line, line + 1):
            got = gpu_encode_all_outputs(gt, bits, mode=P.CNR_RANGE_GREEDY, greedy=params, row_ids=None, n=n)
            pos = np.unique(np.concatenate([np.arange(min(40, n)), np.arange(max(0, n - 40), n), where[where < n], rng.integers(0, n, size=1500)]))
            ora = O.quantize_rows(gt.host[pos], None, bits, mode=O.RANGE_GREEDY, num_bins=params[0], ratio=params[1], n_threads=8)
            compare_greedy(gt.host[pos], {k: got[k][pos] for k in ("scale", "bias", "row_min", "row_max", "codes")}, ora, bits, *params,
                           what="greedy short b%d d%d n%d" % (bits, dim, n))
            assert np.array_equal(got["packed"], O.pack(got["codes"], bits))
    _poll(ctx)


@pytest.mark.parametrize("dim,bits", [(96, 3), (24, 4), (48, 2), (300, 8)])
def test_greedy_skips_ids_outside_the_table(ctx, dim, bits):
    n_rows, n = 500, 133
    table = synth.table_outlier_mix(n_rows, dim, 0.02, 9, DEV)
    ids = _ids(n_rows, n, 3)
    bad = [0, 1, 63, n - 1]
    for k in bad:
        ids[k] = n_rows + k
    prb = P.cnr_packed_row_bytes(dim, bits)
    out = [torch.full((n, w), 0x5A, dtype=torch.uint8, device=DEV) for w in (4, 4, prb)]
    P.cnr_quantize_rows(ctx, table, n_rows, dim, ids, None, n, bits, P.CNR_RANGE_GREEDY, (10, 1.0), out[0].view(torch.float32).reshape(-1),
                        out[1].view(torch.float32).reshape(-1), packed=out[2].reshape(-1))
    _poll(ctx, P.CNR_FLAG_ROW_ID)
    keep = [k for k in range(n) if k not in bad]
    for o in out:
        assert bool((o[bad] == 0x5A).all()) and bool((o[keep] != 0x5A).any(1).all())


# rows of NaN alone, outside the contract: every form reports NaN as their range, scale and bias, and leaves the rows beside them alone
@pytest.mark.parametrize("dim,bits", [(8, 4), (16, 3), (24, 2), (32, 4), (48, 8), (64, 2), (96, 3), (128, 4), (200, 2), (256, 8), (280, 4), (320, 3), (1088, 4)])
def test_greedy_reports_rows_of_nan(ctx, dim, bits):
    print("case greedy nan dim=%d bits=%d" % (dim, bits), flush=True)
    rng = np.random.default_rng(dim)
    rows = rng.normal(0, 0.1, (120, dim)).astype(np.float32)
    bad = np.arange(0, 120, 7)
    with_nan = rows.copy()
    with_nan[bad] = np.nan
    for copies in (1, 500 if dim <= 320 else 200):   # two groups of lanes per row, and one
        want, got = (gpu_encode_all_outputs(GpuTable(ctx, torch.from_numpy(r).to(DEV).repeat(copies, 1)), bits, mode=P.CNR_RANGE_GREEDY, greedy=(20, 1.0),
                                            row_ids=None, n=120 * copies) for r in (rows, with_nan))
        nan_rows = (np.arange(0, 120 * copies, 120)[:, None] + bad).ravel()
        for k in ("scale", "bias", "row_min", "row_max"):
            assert np.isnan(got[k][nan_rows]).all(), (k, got[k][nan_rows][:4])
        rest = np.setdiff1d(np.arange(120 * copies), nan_rows)
        for k in ("scale", "bias", "row_min", "row_max", "codes", "packed"):
            assert np.array_equal(got[k][rest], want[k][rest]), k
    _poll(ctx)


def _early_end_rows(n, dim, bins, seed):
    """Rows whose search may end early, or must not, kind by kind, so that most waves hold one kind and stop when it is finished: a few far
    elements (the best range comes late), both ends far, two clusters (clipping hurts at once), equal elements but one, a range
    small against its offset (down to the narrowest that is searched without divisions), values on the grid, scales over 2**120,
    a skewed density, a log-normal one.  The last row is constant, the one before it too narrow for the fast sequence."""
    rng = np.random.default_rng(seed)
    x = np.empty((n, dim), dtype=np.float64)
    for i in range(n):
        kind, v = i * 9 // n, rng.normal(0, 1, dim)
        if kind == 0:
            v[rng.integers(0, dim, max(1, dim // 64))] = rng.uniform(5, 200) * rng.choice([-1, 1])
        elif kind == 1:
            v[0], v[-1] = rng.uniform(3, 50), -rng.uniform(3, 50)
        elif kind == 2:
            v = rng.choice([-1.0, 1.0], dim) + 0.01 * v
        elif kind == 3:
            v = np.full(dim, 0.5)
            v[rng.integers(dim)] = rng.normal()
        elif kind == 4:
            v = rng.random(dim)
            v[:2] = 0, 1
            v = 1.25 + rng.uniform(1.1, 4) * bins ** 2 * 2.0 ** -23 * v
        elif kind == 5:
            v = rng.integers(0, 4, dim).astype(np.float64)
        elif kind == 6:
            v *= 2.0 ** rng.integers(-60, 61)
        elif kind == 7:
            v = rng.random(dim) ** 8
        else:
            v = np.exp(2 * v)
        x[i] = v * 0.1
    x = x.astype(np.float32)
    x[-1], x[-2] = 0.25, 0.25
    x[-2, 0] = np.nextafter(np.float32(0.25), np.float32(1))
    return x


# The range is the one that the whole search ends with, bit for bit: how far a row is searched depends on the rows that share its wave,
# so the same rows in two orders, kind by kind and mixed, are searched to different ends and have to come out the same.
@pytest.mark.parametrize("dim,bits,bins,long", [(16, 2, 25, 0), (32, 3, 45, 262_144), (64, 4, 100, 131_072), (64, 2, 100, 131_072), (64, 8, 20, 0),
                                                (128, 3, 25, 65_536), (256, 2, 45, 32_768), (256, 4, 45, 0), (8, 4, 45, 49_152),
                                                (96, 2, 45, 26_624), (96, 3, 25, 0), (200, 4, 45, 64_000), (320, 3, 45, 6_400), (1088, 2, 25, 0),
                                                (16, 3, 45, 40_000), (64, 8, 100, 131_072), (128, 4, 45, 65_536), (48, 4, 45, 24_576), (140, 8, 45, 10_700)])
def test_greedy_search_that_ends_early_finds_the_same_range(ctx, dim, bits, bins, long):
    print("case greedy early end dim=%d bits=%d bins=%d" % (dim, bits, bins), flush=True)
    n = 900 if dim <= 320 else 300
    rows = _early_end_rows(n, dim, bins, dim + bits)
    ora = O.quantize_rows(rows, None, bits, mode=O.RANGE_GREEDY, num_bins=bins, ratio=1.0, n_threads=8)
    table = torch.from_numpy(rows).to(DEV)
    keys = ("scale", "bias", "row_min", "row_max", "codes")
    for copies in {1, -(-long // n)} - {0}:   # short lists and those of the long forms
        m = copies * n
        order = np.random.default_rng(m).permutation(m)
        kinds, mixed = (gpu_encode_all_outputs(GpuTable(ctx, t), bits, mode=P.CNR_RANGE_GREEDY, greedy=(bins, 1.0), row_ids=None, n=m)
                        for t in (table.repeat(copies, 1), table[torch.from_numpy(order % n).to(DEV)]))
        for at in {0, m - n}:
            compare_greedy(rows, {k: kinds[k][at:at + n] for k in keys}, ora, bits, bins, 1.0, what="early end b%d d%d n%d" % (bits, dim, m))
        # but for the rows that share a wave (of at most 64) with one searched by division, in either order
        divided = np.zeros((2, m), dtype=bool)
        for o, at in ((0, np.arange(m)), (1, order)):
            hit = np.flatnonzero(at % n == n - 2)
            for k in hit:
                divided[o, k // 64 * 64:k // 64 * 64 + 64] = True
        place = np.empty(m, dtype=np.int64)
        place[order] = np.arange(m)
        keep = ~divided[0] & ~divided[1][place]
        assert keep.mean() > 0.75 or m == n
        for k in keys + ("packed",):
            assert np.array_equal(kinds[k][keep], mixed[k][place[keep]]), k
    _poll(ctx)


# Lists whose length only the device knows, in buffers that may hold long ones: one launch has both forms.  On either side of the line, empty, of one row, and
# longer than the buffers; whole searches and partial ones.  The same rows with the length known to the host have to come out the same.
@pytest.mark.parametrize("dim,bits,line", [(8, 4, 24_576), (24, 3, 49_152), (32, 2, 262_144), (40, 2, 24_576), (64, 4, 131_072), (64, 8, 131_072), (96, 3, 26_624), (128, 2, 65_536),
                                           (140, 8, 10_649), (140, 4, 26_624), (256, 3, 32_768), (200, 4, 64_000)])
def test_greedy_lists_of_a_length_that_only_the_device_knows(ctx, dim, bits, line):
    cap = line * 5 // 4
    table = synth.table_outlier_mix(cap, dim, 0.02, dim + bits, DEV)
    ids = _ids(cap, cap, 3)
    for bins, ratio in ((20, 1.0), (20, 0.15)):
        out = {}
        for n, known in ((cap, True), (0, False), (1, False), (777, False), (line - 1, False), (line, False), (cap + 5, False)):
            sc, bi = torch.full((cap,), -7.0, device=DEV), torch.full((cap,), -7.0, device=DEV)
            pk = torch.full((cap * P.cnr_packed_row_bytes(dim, bits),), 77, dtype=torch.uint8, device=DEV)
            n_dev = None if known else torch.tensor([n], dtype=torch.int64, device=DEV)
            P.cnr_quantize_rows(ctx, table, cap, dim, ids, n_dev, cap, bits, P.CNR_RANGE_GREEDY, (bins, ratio), sc, bi, packed=pk)
            if known:
                out = dict(scale=sc, bias=bi, packed=pk.reshape(cap, -1))
                continue
            live = min(n, cap)
            assert torch.equal(sc[:live], out["scale"][:live]) and torch.equal(bi[:live], out["bias"][:live]), n
            assert torch.equal(pk.reshape(cap, -1)[:live], out["packed"][:live]), n
            assert (sc[live:] == -7.0).all() and (bi[live:] == -7.0).all() and (pk.reshape(cap, -1)[live:] == 77).all(), n
    _poll(ctx)


# At 8 bits the question is asked before the first iteration too: a step of many codes, of about one, of less than one, and a search of one step.
@pytest.mark.parametrize("dim,n", [(16, 900), (24, 900), (64, 900), (64, 131_400), (96, 10_800), (256, 900), (320, 900), (1088, 300)])
@pytest.mark.parametrize("bins,ratio", [(2, 1.0), (20, 0.05), (20, 1.0), (200, 1.0), (400, 0.2)])
def test_greedy_search_at_8_bits_that_ends_before_it_starts(ctx, dim, n, bins, ratio):
    some = min(n, 900)
    rows = _early_end_rows(some, dim, bins, dim + bins)
    ora = O.quantize_rows(rows, None, 8, mode=O.RANGE_GREEDY, num_bins=bins, ratio=ratio, n_threads=8)
    gt = GpuTable(ctx, torch.from_numpy(rows).to(DEV).repeat(n // some, 1))
    got = gpu_encode_all_outputs(gt, 8, mode=P.CNR_RANGE_GREEDY, greedy=(bins, ratio), row_ids=None, n=n)
    keys = ("scale", "bias", "row_min", "row_max", "codes")
    for at in {0, n - some}:
        compare_greedy(rows, {k: got[k][at:at + some] for k in keys}, ora, 8, bins, ratio, what="8 bits d%d n%d bins%d" % (dim, n, bins))
    _poll(ctx)


# Partial searches up to 0.52, 0.32 and 0.18 of their moves (2, 3, 4 bits) go through kernels that do not ask whether a row is finished
@pytest.mark.parametrize("dim,bits,long", [(36, 2, 25_000), (40, 3, 25_000), (64, 2, 131_072), (64, 4, 131_072), (96, 4, 26_624), (128, 3, 65_536), (200, 3, 64_000),
                                           (256, 2, 32_768), (280, 4, 0), (320, 4, 6_400), (1088, 2, 0), (32, 4, 262_144), (8, 3, 49_152)])
def test_greedy_partial_searches(ctx, dim, bits, long):
    last = {2: 26, 3: 16, 4: 9}[bits]
    for n in {300, max(300, long + 3)}:
        gt = GpuTable(ctx, synth.table_outlier_mix(n, dim, 0.02, dim + bits, DEV))
        pos = np.unique(np.concatenate([np.arange(200), np.random.default_rng(n).integers(0, n, size=1000), [n - 1]]))
        for n_iter in (last, last + 1):
            ratio = (n_iter - 0.5) / 50
            assert P.cnr_greedy_iterations(50, ratio) == n_iter
            got = gpu_encode_all_outputs(gt, bits, mode=P.CNR_RANGE_GREEDY, greedy=(50, ratio), row_ids=None, n=n)
            ora = O.quantize_rows(gt.host[pos], None, bits, mode=O.RANGE_GREEDY, num_bins=50, ratio=ratio, n_threads=8)
            compare_greedy(gt.host[pos], {k: got[k][pos] for k in ("scale", "bias", "row_min", "row_max", "codes")}, ora, bits, 50, ratio,
                           what="partial b%d d%d n%d" % (bits, dim, n))
            assert np.array_equal(got["packed"], O.pack(got["codes"], bits))
    _poll(ctx)


# A row without an error from the start (here constant) is finished: it must not keep the rows that share its wave searching.  Measured, the
# result is the same either way: with one such row in 64 the long lists took 1.2 to 4 times as long.
@pytest.mark.parametrize("dim,bits,bins,n", [(64, 4, 100, 300_000), (16, 4, 45, 600_000), (24, 4, 45, 400_000), (48, 4, 100, 300_000), (128, 4, 100, 150_000)])
def test_constant_rows_do_not_keep_a_search_going(ctx, dim, bits, bins, n):
    print("case greedy constant rows dim=%d" % dim, flush=True)
    prb = P.cnr_packed_row_bytes(dim, bits)
    tables = [synth.table_outlier_mix(n, dim, 0.02, 5, DEV) for _ in range(2)]
    tables[1][::64] = 0.25
    outs = [(torch.empty(n, device=DEV), torch.empty(n, device=DEV), torch.empty(n * prb, dtype=torch.uint8, device=DEV)) for _ in range(2)]
    best = [float("inf")] * 2
    for _ in range(7):
        for i, (t, (scale, bias, packed)) in enumerate(zip(tables, outs)):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            P.cnr_quantize_rows(ctx, t, n, dim, None, None, n, bits, P.CNR_RANGE_GREEDY, (bins, 1.0), scale, bias, packed=packed)
            end.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], start.elapsed_time(end))
    print("without %.3f ms, with %.3f" % tuple(best), flush=True)
    assert best[1] < 1.5 * best[0]
    others = torch.arange(n, device=DEV) % 64 != 0
    for a, b in zip(*outs):
        assert torch.equal(a.view(n, -1)[others], b.view(n, -1)[others])
    assert bool((outs[1][0][::64] == 0).all()) and bool((outs[1][1][::64] == 0.25).all())
    _poll(ctx)


# Exact ties: with qmax + 1 bins a step is one code step at the first move already, at 3 bits and 12 bins
# after five (7 / (12 - 5) = 1), and these rows have nothing but their two ends beyond the bounds then; the
# setting is the one whose tie lies at the best range of the row length (1 row in 100 to 1000).
@pytest.mark.parametrize("dim,bits,bins,n,piece", [
    (16, 2, 4, 60_000, 20_000), (64, 3, 8, 140_000, 12_000), (64, 3, 8, 140_000, 70_000), (256, 3, 12, 34_000, 6_000), (256, 3, 12, 34_000, 17_000),
    (24, 2, 4, 60_000, 20_000), (48, 2, 4, 60_000, 20_000), (96, 3, 8, 60_000, 15_000), (200, 3, 12, 90_000, 15_000), (272, 3, 12, 24_000, 3_000),
    (320, 3, 12, 24_000, 3_000)])
def test_greedy_ranges_do_not_depend_on_the_list_length(ctx, dim, bits, bins, n, piece):
    print("case greedy ties dim=%d n=%d piece=%d" % (dim, n, piece), flush=True)
    g = torch.Generator(device=DEV).manual_seed(dim)
    table = torch.empty(n, dim, device=DEV).normal_(0, 0.02, generator=g)
    for half, sign in ((0, 1.0), (dim // 2, -1.0)):
        col = half + torch.randint(0, dim // 2, (n,), generator=g, device=DEV)
        table[torch.arange(n, device=DEV), col] = torch.empty(n, device=DEV).uniform_(0.1, 0.12, generator=g) * sign
    prb = P.cnr_packed_row_bytes(dim, bits)

    def encode(parts):
        scale, bias, packed = torch.empty(n, device=DEV), torch.empty(n, device=DEV), torch.empty(n * prb, dtype=torch.uint8, device=DEV)
        for a, b in parts:   # whole multiples of 16 rows: aligned pieces of the buffers
            P.cnr_quantize_rows(ctx, table[a:b], b - a, dim, None, None, b - a, bits, P.CNR_RANGE_GREEDY, (bins, 1.0), scale[a:b], bias[a:b],
                                packed=packed[a * prb:b * prb])
        return scale, bias, packed

    piece &= ~15
    whole = encode([(0, n)])
    for w, p, what in zip(whole, encode([(a, min(n, a + piece)) for a in range(0, n, piece)]), ("scale", "bias", "packed")):
        assert torch.equal(w, p), "%s: %d of %d differ" % (what, int((w != p).sum()), w.numel())
    pos = np.arange(0, n, max(1, n // 6000))
    rows = table[torch.from_numpy(pos).to(DEV)].cpu().numpy()
    ora = O.quantize_rows(rows, None, bits, mode=O.RANGE_GREEDY, num_bins=bins, ratio=1.0, n_threads=8)
    got = dict(scale=whole[0].cpu().numpy()[pos], bias=whole[1].cpu().numpy()[pos], row_min=ora["row_min"], row_max=ora["row_max"],
               codes=O.unpack(whole[2].view(n, prb)[torch.from_numpy(pos).to(DEV)].cpu().numpy(), dim, bits))
    ties = compare_greedy(rows, got, ora, bits, bins, 1.0, what="greedy ties d%d" % dim)
    print("rows whose tie the oracle decided by rounding: %d" % ties, flush=True)
    _poll(ctx)


# ---- min/max and symmetric ranges at row lengths that are no power of two: every shape's first and last -

@pytest.mark.parametrize("dim,bits", [
    (4, 2), (8, 3), (12, 8), (20, 4), (28, 2), (36, 4), (40, 3), (48, 8), (52, 2), (60, 4), (72, 3), (96, 8), (100, 2),
    (120, 3), (132, 4), (160, 3), (164, 8), (192, 2), (196, 4), (224, 3), (228, 2), (252, 8), (260, 2), (320, 3), (324, 4),
    (384, 8), (388, 2), (448, 3), (452, 4), (512, 8), (516, 2), (1000, 3)])
def test_encode_of_other_row_lengths(ctx, dim, bits):
    print("case units dim=%d bits=%d" % (dim, bits), flush=True)
    n_rows = 1300
    table = synth.table_normal(n_rows, dim, 0.05, dim, DEV)
    special = _special_rows(dim, dim)
    table[torch.arange(special.shape[0], device=DEV) * 61 + 3] = torch.from_numpy(special).to(DEV)
    gt = GpuTable(ctx, table)
    for mode, ora_mode in ((P.CNR_RANGE_MINMAX, O.RANGE_MINMAX), (P.CNR_RANGE_SYMMETRIC, O.RANGE_SYMMETRIC)):
        for n in (1, 16, 63, 257, 1300):      # rows 0 .. n-1, and a list known on the device alone
            got = gpu_encode_all_outputs(gt, bits, mode=mode, row_ids=None, n=n)
            compare_quantized(gt.host[:n], got, O.quantize_rows(gt.host[:n], None, bits, mode=ora_mode), bits, what="units d%d n%d" % (dim, n))
            assert np.array_equal(got["packed"], O.pack(got["codes"], bits))
        ids = np.flatnonzero(np.random.default_rng(dim).random(n_rows) < 0.4)
        gt.ck.clear()
        gt.ck.mark(torch.from_numpy(ids).to(DEV))
        gt.ck.compact()
        got = gpu_encode_all_outputs(gt, bits, mode=mode)
        assert got["n"] == ids.size
        compare_quantized(gt.host[ids], got, O.quantize_rows(gt.host, ids.astype(np.uint32), bits, mode=ora_mode), bits, what="units d%d list" % dim)
        assert np.array_equal(got["packed"], O.pack(got["codes"], bits))
    _poll(ctx)


# short lists go a row (or several short ones) per wave; `short` is the longest of them, of every shape
@pytest.mark.parametrize("dim,bits,short", [
    (4, 2, 98_304), (12, 8, 98_304), (20, 4, 49_152), (24, 3, 49_152), (36, 4, 24_576), (40, 3, 24_576), (48, 8, 24_576), (52, 2, 24_576),
    (60, 4, 24_576), (72, 3, 12_288), (96, 8, 12_288), (100, 2, 12_288), (120, 3, 12_288), (132, 4, 6_144), (160, 3, 6_144), (164, 8, 6_144),
    (192, 2, 6_144), (196, 4, 12_288), (224, 3, 12_288), (228, 2, 12_288), (252, 8, 12_288), (260, 2, 12_288), (320, 3, 12_288),
    (324, 4, 16_384), (384, 8, 16_384), (388, 2, 32_768), (448, 3, 32_768), (452, 4, 65_536), (512, 8, 65_536)])
def test_encode_of_other_row_lengths_on_either_side_of_a_short_list(ctx, dim, bits, short):
    print("case short units dim=%d bits=%d" % (dim, bits), flush=True)
    n = short + 21
    gt = GpuTable(ctx, synth.table_normal(n, dim, 0.05, dim, DEV))
    for mode, ora_mode in ((P.CNR_RANGE_MINMAX, O.RANGE_MINMAX), (P.CNR_RANGE_SYMMETRIC, O.RANGE_SYMMETRIC)):
        long = gpu_encode_all_outputs(gt, bits, mode=mode, row_ids=None, n=n)
        pos = np.unique(np.concatenate([np.arange(min(n, 300)), np.arange(n - 300, n), np.random.default_rng(dim).integers(0, n, size=4000)]))
        ora = O.quantize_rows(gt.host[pos], None, bits, mode=ora_mode, n_threads=8)
        compare_quantized(gt.host[pos], {k: long[k][pos] for k in ("scale", "bias", "row_min", "row_max", "codes")}, ora, bits, what="long d%d" % dim)
        assert np.array_equal(long["packed"], O.pack(long["codes"], bits))
        some = gpu_encode_all_outputs(gt, bits, mode=mode, row_ids=None, n=short)
        # the capacity allows a long list, the device's count is a short or a long one
        gt.ck.row_ids.copy_(torch.arange(n, dtype=torch.int32, device=DEV))
        for got, m in [(some, short)] + [(None, m) for m in (0, 17, min(short, 6_000), n - 3)]:
            if got is None:
                gt.ck.n_dirty.fill_(m)
                got = gpu_encode_all_outputs(gt, bits, mode=mode)
            for k in ("scale", "bias", "row_min", "row_max", "codes", "packed"):
                assert np.array_equal(got[k], long[k][:m]), (k, m)
    _poll(ctx)


@pytest.mark.parametrize("dim,bits,n", [(8, 3, 133), (20, 2, 133), (96, 4, 133), (144, 8, 133), (500, 4, 133), (516, 2, 133),
                                        (8, 3, 98_400), (20, 2, 49_200), (96, 4, 12_300), (144, 8, 6_200), (320, 3, 12_300)])
def test_encode_of_other_row_lengths_skips_ids_outside_the_table(ctx, dim, bits, n):
    n_rows = n + 367
    table = synth.table_normal(n_rows, dim, 0.05, 9, DEV)
    ids = _ids(n_rows, n, 3)
    prb = P.cnr_packed_row_bytes(dim, bits)

    def encode(ids):
        out = [torch.full((n, w), 0x5A, dtype=torch.uint8, device=DEV) for w in (4, 4, prb, dim)]
        P.cnr_quantize_rows(ctx, table, n_rows, dim, ids, None, n, bits, P.CNR_RANGE_MINMAX, None, out[0].view(torch.float32).reshape(-1),
                            out[1].view(torch.float32).reshape(-1), codes_u8=out[3].reshape(-1), packed=out[2].reshape(-1))
        return out

    whole = encode(ids)
    _poll(ctx)
    bad = [0, 1, 63, n - 1]
    for k in bad:
        ids[k] = n_rows + k
    some = encode(ids)
    _poll(ctx, P.CNR_FLAG_ROW_ID)
    keep = [k for k in range(n) if k not in bad]
    for w, o in zip(whole, some):             # nothing of theirs is written, everything else as without them
        assert bool((o[bad] == 0x5A).all()) and torch.equal(o[keep], w[keep])


# ---- parameter selection: lanes per row, sets of parameters per launch, partial sums that fit the scratch --

@pytest.mark.parametrize("dim,bits,n,bins", [
    (64, 3, 1, tuple(range(2, 42))),       # a scratch of ten sums: several launches per grid
    (64, 4, 301, tuple(range(3, 40))),     # more points than a launch takes
    (64, 2, 44_000, (7, 20)), (96, 3, 43_691, (9, 16)), (200, 4, 43_800, (18, 30)),   # four lanes per row
    (96, 4, 500, (18, 30)), (284, 2, 77, (9, 12)), (288, 8, 77, (9, 12)),              # twice eight, twice thirty-two
    (1148, 2, 130, (8, 11)), (1152, 3, 65, (9, 12)), (4, 8, 40, (3, 20)), (32, 3, 300, (9, 12)),   # the same, sixty-four; twice four
])
def test_parameter_selection_routes(ctx, dim, bits, n, bins):
    print("case select dim=%d bits=%d n=%d" % (dim, bits, n), flush=True)
    n_rows, ratios = n + 50, (0.25, 0.5, 1.0)
    table = synth.table_outlier_mix(n_rows, dim, 0.02, dim + n, DEV)
    table[3] = 0.25                        # a constant row: searched by division
    ids = _ids(n_rows, n, 11)
    choice, report = P.select_greedy_params(ctx, table, n_rows, dim, ids, bits, bins, ratios)
    rows = table[ids.long()].cpu().numpy()
    want = {"naive": O.mean_l2(rows, bits, O.RANGE_MINMAX)}
    scale, bias = torch.empty(n, device=DEV), torch.empty(n, device=DEV)
    packed = torch.empty(n * P.cnr_packed_row_bytes(dim, bits), dtype=torch.uint8, device=DEV)
    err = torch.empty(n, dtype=torch.float64, device=DEV)
    for key, num_bins, ratio in [(("bins", b), b, 1.0) for b in bins] + [(("ratio", r), choice[0], r) for r in ratios]:
        # the oracle's errors, but for the rows whose exact tie it decides by rounding: there the encoder's
        ora = O.quantize_rows(rows, None, bits, mode=O.RANGE_GREEDY, num_bins=num_bins, ratio=ratio, n_threads=8)
        errors = O.row_l2(rows, O.dequantize(ora["codes"], ora["scale"], ora["bias"]))[0].copy()
        P.cnr_quantize_rows(ctx, table, n_rows, dim, ids, None, n, bits, P.CNR_RANGE_GREEDY, (num_bins, ratio), scale, bias, packed=packed)
        P.cnr_quant_error(ctx, table, n_rows, dim, ids, None, n, bits, packed, scale, bias, err)
        tied = tie_rows(rows, dict(scale=scale.cpu().numpy(), bias=bias.cpu().numpy()), ora, bits, num_bins, ratio)
        errors[tied] = err.cpu().numpy()[tied]
        want[key] = float(errors.mean())
    assert set(report) == set(want)
    for key in want:                       # fp64 sums in another order
        assert report[key] == pytest.approx(want[key], rel=1e-9), key
    num_bins = O.taper_choice(list(bins), [want[("bins", b)] for b in bins], want["naive"], 0.05)
    assert choice == (num_bins, O.taper_choice(list(ratios), [want[("ratio", r)] for r in ratios], want["naive"], 0.05))
    _poll(ctx)


# Points that share a search: grids in any order, values twice, no ratio 1, ratios without an iteration, one stop only; in one launch (up to 32 points that fit the
# scratch) and in two, whose ratios are searched apart or (many rows) together; launches in which a wave takes several passes (4096 workgroups).
@pytest.mark.parametrize("dim,bits,n,bins,ratios", [
    (64, 3, 700, (45, 10, 25, 10), (1.0, 0.3, 0.6, 0.3)),
    (36, 2, 300, (25, 9, 45, 16), (0.2, 0.0, 0.6)),
    (40, 2, 500, (12, 30), (0.0,)), (96, 4, 130, (30, 30), (1.0,)), (288, 2, 257, (20, 8, 14, 11), (0.7, 0.2)),
    (16, 4, 900, (2, 1, 40), (0.5, 1.5, 0.05)), (144, 2, 1001, (1,), (0.4, 0.0, 0.9)),
    (64, 2, 300, (40, 3, 22, 3, 17, 9, 30, 12, 5, 26, 33), (0.8, 0.25, 0.5)), (24, 8, 90_000, tuple(range(13, 2, -1)), (0.9, 0.0, 0.3)),
    (8, 4, 262_500, (9, 3), (0.6, 0.3)), (32, 4, 2, (14, 6), (0.5, 0.9)), (64, 4, 5, (14, 6), (0.5, 0.9)),
])
def test_parameter_selection_with_shared_searches(ctx, dim, bits, n, bins, ratios):
    print("case select dim=%d bits=%d n=%d" % (dim, bits, n), flush=True)
    table = synth.table_outlier_mix(n, dim, 0.02, dim + n, DEV)
    table[1] = 0.25                        # searched by division
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    choice, report = P.select_greedy_params(ctx, table, n, dim, ids, bits, bins, ratios)
    rows = table.cpu().numpy()
    scale, bias = torch.empty(n, device=DEV), torch.empty(n, device=DEV)
    packed = torch.empty(n * P.cnr_packed_row_bytes(dim, bits), dtype=torch.uint8, device=DEV)
    err = torch.empty(n, dtype=torch.float64, device=DEV)

    def mean(num_bins, ratio):             # the oracle's, but for the rows whose exact tie it decides by rounding: there the encoder's
        ora = O.quantize_rows(rows, None, bits, mode=O.RANGE_GREEDY, num_bins=num_bins, ratio=ratio, n_threads=8)
        errors = O.row_l2(rows, O.dequantize(ora["codes"], ora["scale"], ora["bias"]))[0].copy()
        P.cnr_quantize_rows(ctx, table, n, dim, ids, None, n, bits, P.CNR_RANGE_GREEDY, (num_bins, ratio), scale, bias, packed=packed)
        P.cnr_quant_error(ctx, table, n, dim, ids, None, n, bits, packed, scale, bias, err)
        tied = tie_rows(rows, dict(scale=scale.cpu().numpy(), bias=bias.cpu().numpy()), ora, bits, num_bins, ratio)
        errors[tied] = err.cpu().numpy()[tied]
        return float(errors.mean())

    want = {"naive": O.mean_l2(rows, bits, O.RANGE_MINMAX)}
    want.update({("bins", b): mean(b, 1.0) for b in bins})
    assert choice[0] == O.taper_choice(list(bins), [want[("bins", b)] for b in bins], want["naive"], 0.05)
    want.update({("ratio", r): mean(choice[0], r) for r in ratios})
    assert set(report) == set(want)
    for key in want:                       # fp64 sums in another order
        assert report[key] == pytest.approx(want[key], rel=1e-9), key
    assert choice[1] == np.float32(O.taper_choice(list(ratios), [want[("ratio", r)] for r in ratios], want["naive"], 0.05))
    _poll(ctx)


# ---- compaction: workgroups that count the tiles before theirs, up to 64 tiles; counted tiles beyond ------

@pytest.mark.parametrize("n_rows", [16_384, 16_385, 8 * 16_384 + 1, 64 * 16_384, 64 * 16_384 + 1])
@pytest.mark.parametrize("shift", [0, 1])
def test_compaction_around_the_self_counting_limit(ctx, n_rows, shift):
    g = torch.Generator(device=DEV).manual_seed(n_rows)
    words = P.cnr_bitmap_words(n_rows)
    bitmap = torch.randint(-2**31, 2**31, (words + shift,), generator=g, device=DEV).to(torch.int32)[shift:]
    bits = ((bitmap[:, None] >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1).reshape(-1)[:n_rows]   # bits past n_rows are set too
    want = torch.nonzero(bits).reshape(-1).to(torch.int32)
    scratch = torch.empty((P.cnr_scratch_bytes(n_rows) + 7) // 8, dtype=torch.int64, device=DEV)
    for capacity in (n_rows, want.numel() - 5):
        ids = torch.full((n_rows,), -1, dtype=torch.int32, device=DEV)
        n = torch.zeros(1, dtype=torch.int64, device=DEV)
        P.cnr_compact_dirty(ctx, bitmap, n_rows, ids, capacity, n, scratch)
        assert int(n) == want.numel()
        m = min(capacity, want.numel())
        assert torch.equal(ids[:m], want[:m]) and bool((ids[m:] == -1).all())
        _poll(ctx, 0 if capacity >= want.numel() else P.CNR_FLAG_CAPACITY)


@pytest.mark.parametrize("tables,tiles", [(9, 64), (10, 64), (16, 48), (16, 49)])
def test_batched_compaction_around_the_self_counting_limit(ctx, tables, tiles):
    # what a launch's workgroups count themselves grows with its tables; they differ in size and share nothing
    cks, wants = [], []
    for k in range(tables):
        n_rows = tiles * 16_384 - (7 * k if k else 0)
        ck = P.TableCheckpointer(ctx, n_rows, 8, device=DEV)
        g = torch.Generator(device=DEV).manual_seed(k)
        ck.bitmap.copy_(torch.randint(-2**31, 2**31, (ck.bitmap.numel(),), generator=g, device=DEV).to(torch.int32))
        bits = ((ck.bitmap[:, None] >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1).reshape(-1)[:n_rows]
        wants.append(torch.nonzero(bits).reshape(-1).to(torch.int32))
        ck.row_ids.fill_(-1)
        cks.append(ck)
    P.BatchCheckpointer(ctx, cks).compact()
    for ck, want in zip(cks, wants):
        n = int(ck.n_dirty)
        assert n == want.numel() and torch.equal(ck.row_ids[:n], want) and bool((ck.row_ids[n:] == -1).all())
    _poll(ctx)


# ---- bulk mark of one-slice tables: streams from 64 MB on are read past the caches -------------------------

# Long streams of a batch: slices in two to thirty-two parts of the streams, or flag bytes, by what the call's tables come to; tables of one and several
# slices, of different sizes, some of whose scratch has room for eight parts only.
@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
@pytest.mark.parametrize("tables,n_rows,n_idx", [(16, 1_310_720, 70_661), (16, 5_000_003, 85_100), (8, 1_310_721, 131_073), (8, 400_001, 524_289), (8, 1_000_003, 1_500_000),
                                                 (4, 1_310_719, 3_000_001), (2, 4_000_000, 2_000_001), (1, 1_310_720, 9_000_001), (1, 777_777, 70_001), (3, 200_033, 150_000)])
def test_bulk_mark_of_a_batch_in_parts(ctx, dtype, tables, n_rows, n_idx):
    rng = np.random.default_rng(tables + n_idx)
    g = torch.Generator(device=DEV).manual_seed(n_idx)
    rows = [n_rows if i % 3 == 0 else max(66, n_rows // (i % 5 + 1) - i) for i in range(tables)]
    scratch = [P.TableCheckpointer.new_mark_scratch(n, DEV) for n in rows]
    cks = [P.TableCheckpointer(ctx, n, 64, device=DEV, mark_scratch=m) for n, m in zip(rows, scratch)]
    batch = P.BatchCheckpointer(ctx, cks)
    batch.clear()
    want, skipped = [torch.zeros(n + 64, dtype=torch.bool, device=DEV) for n in rows], 0
    for call in range(2):
        streams = []
        for t, n in enumerate(rows):
            u = torch.rand(n_idx + int(rng.integers(0, 9)), generator=g, device=DEV, dtype=torch.float64)
            idx = ((u ** 3 * (n + 3)).long() - 1)[int(rng.integers(0, 3)):]   # skewed; -1, n and n + 1 are outside
            idx[-1], idx[0] = n - 1, 0
            good = (idx >= 0) & (idx < n)
            want[t][idx[good]] = True
            skipped += int((~good).sum())
            streams.append(idx.to(dtype))
        batch.mark(streams)
    for t, n in enumerate(rows):
        bits = ((cks[t].bitmap[:, None] >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1).reshape(-1)[:n]
        assert torch.equal(bits.bool(), want[t][:n]), (t, n)
        assert not scratch[t].any()
    _, bad, _ = P.cnr_poll_errors(ctx)
    assert bad == skipped


# Short streams: a workgroup's look-ups of one row agree on one of them (by the top twelve bits of row * 0x9E3779B1).  Repeats of few rows, of
# rows that meet in one place there, and none, at the edges of a workgroup's 1024 look-ups and over several passes (2048 workgroups).
@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
@pytest.mark.parametrize("n_rows", [1, 33, 200_001, 2_200_000_000])
@pytest.mark.parametrize("n_idx", [1, 255, 1_024, 1_025, 65_537, 2_097_153 + 1_030])
def test_short_mark_with_repeats(ctx, dtype, n_rows, n_idx):
    reach = min(n_rows, 2**31 - 1) if dtype is torch.int32 else n_rows
    rng = np.random.default_rng(n_rows % 1000 + n_idx)
    place = (np.arange(min(reach, 200_000), dtype=np.uint64) * 0x9E3779B1 % 2**32) >> 20
    together = np.flatnonzero(place == place[-1])
    few = np.concatenate([together[:40], rng.integers(0, reach, 9), [reach - 1]])
    bitmap = torch.zeros(P.cnr_bitmap_words(n_rows), dtype=torch.int32, device=DEV)
    for stream in (few[rng.integers(0, len(few), n_idx)], rng.integers(0, reach, n_idx)):
        stream = stream.astype(np.int64)
        out = rng.random(n_idx) < 0.01
        stream[out] = rng.choice([-1, -2**31] + ([n_rows] if n_rows < 2**31 else [2**31 - 1]), int(out.sum()))
        want = np.unique(stream[(stream >= 0) & (stream < n_rows)])
        P.cnr_clear_bitmap(ctx, bitmap, n_rows)
        P.cnr_mark_touched(ctx, bitmap, n_rows, torch.from_numpy(stream).to(DEV).to(dtype))
        words = torch.nonzero(bitmap).reshape(-1)
        bits = np.unpackbits(bitmap[words].cpu().numpy().view(np.uint8).reshape(-1, 4), axis=1, bitorder="little")
        got = (words.cpu().numpy()[:, None] * 32 + np.arange(32))[bits == 1]
        assert np.array_equal(got, want)
        _, bad, _ = P.cnr_poll_errors(ctx)
        assert bad == int(((stream < 0) | (stream >= n_rows)).sum())


# Waves whose 64 rows ascend set a word's bits with one atomic OR.  Every row, gaps, gaps of over a word, repeats (which do not ascend strictly), descending,
# waves of both kinds in a workgroup, bits set before, ends of the stream within a wave; 64-bit look-ups outside the table that ascend with the others by their
# lower halves, first in a word or not.
@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
@pytest.mark.parametrize("n_idx", [1, 63, 64, 65, 256, 1_024, 4_133, 2_097_152 + 1_105])
def test_short_mark_of_ascending_rows(ctx, dtype, n_idx):
    rng = np.random.default_rng(n_idx)
    k = np.arange(n_idx)
    few = np.sort(rng.choice(5 * n_idx, n_idx, replace=False))
    mixed = np.where((k // 64) % 3 == 1, rng.permutation(few), few)
    streams = [k, 3 * k + 1, 41 * k, few, np.sort(rng.integers(0, 2 * n_idx, n_idx)), few[::-1].copy(), mixed]
    if dtype is torch.int64:
        streams += [k + (rng.random(n_idx) < 0.3) * 2**32, k + (k % 32 == 0) * 2**33, few - (rng.random(n_idx) < 0.05) * 2**40, k + (k % 2 == 0) * 2**32]
    else:
        streams += [np.where(rng.random(n_idx) < 0.02, -1 - k, k)]
    for stream in streams:
        stream = stream.astype(np.int64)
        n_rows = int(max(1, stream[(stream >= 0) & (stream < 2**31)].max(initial=0))) + (1 if n_idx % 2 else -2 if n_idx > 64 else 0)
        good = (stream >= 0) & (stream < n_rows)
        bitmap = torch.zeros(P.cnr_bitmap_words(n_rows), dtype=torch.int32, device=DEV)
        want, bad = np.zeros(32 * bitmap.numel(), dtype=bool), 0
        for part in (stream[::7].copy(), stream, stream[1:].copy()):
            if part.size == 0:
                continue
            part_good = (part >= 0) & (part < n_rows)
            want[part[part_good]] = True
            bad += int((~part_good).sum())
            P.cnr_mark_touched(ctx, bitmap, n_rows, torch.from_numpy(part).to(DEV).to(dtype))
            got = np.unpackbits(bitmap.cpu().numpy().view(np.uint8), bitorder="little").astype(bool)
            assert np.array_equal(got, want), (n_rows, part.size)
        assert P.cnr_poll_errors(ctx)[1] == bad and (good.any() or bad)


def test_marking_rows_in_order_takes_no_longer_than_in_no_order(ctx):
    # the ORs of a list in order meet in few words: 102 us against 77 without anything about that, 5 and 68 with it
    n = 1_000_000
    bitmap = torch.zeros(P.cnr_bitmap_words(n), dtype=torch.int32, device=DEV)
    begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    took = []
    for ids in (torch.arange(n, device=DEV), torch.randperm(n, device=DEV)):
        for timed in (False, True):
            begin.record()
            for _ in range(20):
                P.cnr_clear_bitmap(ctx, bitmap, n)
                P.cnr_mark_touched(ctx, bitmap, n, ids)
            end.record()
            end.synchronize()
        took.append(begin.elapsed_time(end))
    assert took[0] < took[1], took


@pytest.mark.parametrize("dtype,n_idx", [(torch.int64, 1_048_576), (torch.int64, 1_048_577), (torch.int32, 2_097_151), (torch.int32, 2_097_160)])
@pytest.mark.parametrize("n_rows", [1_310_720, 200_001])
def test_bulk_mark_around_the_streaming_limit(ctx, dtype, n_idx, n_rows):
    tables, shift = 8, 3   # the streams start off a 16-byte boundary: head and tail elements
    g = torch.Generator(device=DEV).manual_seed(n_idx)
    cks = [P.TableCheckpointer(ctx, n_rows, 64, capacity=1, device=DEV, mark_scratch=P.TableCheckpointer.new_mark_scratch(n_rows)) for _ in range(tables)]
    idx = [torch.randint(-2, n_rows + 2, (n_idx + shift,), generator=g, device=DEV).to(dtype)[shift:] for _ in range(tables)]
    batch = P.BatchCheckpointer(ctx, cks)
    batch.mark(idx)
    bad = 0
    for ck, t in zip(cks, idx):
        inside = (t >= 0) & (t < n_rows)
        bad += int((~inside).sum())
        want = torch.zeros(32 * ck.bitmap.numel(), dtype=torch.bool, device=DEV)
        want[t[inside].long()] = True
        bits = ((ck.bitmap[:, None] >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1).bool().reshape(-1)
        assert torch.equal(bits, want)
        assert not bool(ck.mark_scratch.any())
    st, n_bad, flags = P.cnr_poll_errors(ctx)
    assert (n_bad, flags) == (bad, 0)


# two groups of sixteen lanes for rows of 144 to 284 elements, up to 8192 rows and sets together
@pytest.mark.parametrize("dim,bits,n", [(140, 2, 300), (144, 3, 257), (200, 2, 1_639), (200, 4, 1_638), (256, 8, 70), (284, 4, 31), (284, 2, 1)])
def test_parameter_selection_of_longer_rows(ctx, dim, bits, n):
    test_parameter_selection_routes(ctx, dim, bits, n, (10, 25, 45, 100))
