"""The dispatch branches of the row kernels at the sizes where they can go wrong: list lengths on either
side of a branch, remainders of lane groups and workgroups, row lengths that are no power of two,
unaligned tables, counts on the device below the capacity, ids outside the table."""
import numpy as np
import pytest
import torch

import paper_2010_08679_amd as P
from paper_2010_08679_amd import synth

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
    (100, 2, 17_001, 0), (96, 3, 33_000, 0), (516, 4, 16_500, 0),                                # several trips, the last one partial
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
    for live in sorted({n, max(1, n - 777), n // 2, 0}):       # the count on the device
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
