"""Products at widths, leading dimensions and offsets off 16 bytes (bspmm_any_kernel): tile rows copied as
the 16-byte words they lie in, a last lane that holds part of a row, a lane per float for long rows,
row blocks; compared with the oracle, with guards around everything that may be written."""
import numpy as np
import pytest

from paper_1903_11409_amd import bspmm as K
from paper_1903_11409_amd import workloads as W

pytestmark = pytest.mark.gpu

SENTINEL = -12345.0
# (rows, cols, entries): one row, one column, more rows than lanes, rows of hundreds of entries, more than
# four entries per lane, nothing, too large for LDS at any width
SHAPES = [(1, 1, 1), (1, 220, 300), (220, 1, 400), (31, 33, 90), (300, 20, 900), (5, 200, 1300), (0, 0, 0), (7, 9, 0),
          (64, 64, 200), (3, 5000, 700), (900, 2500, 2600)]


def _run(torch, plan, b, transposed, in_off, out_off, in_extra, out_extra):
    src, rows = (b.dY, b.n_b_rows) if transposed else (b.B, b.n_c_rows)
    ld_in, ld_out = b.F + in_extra, b.F + out_extra
    store_in = torch.full((src.shape[0] * ld_in + in_off + 4,), float("nan"), device="cuda")
    X = store_in[in_off:in_off + src.shape[0] * ld_in].view(-1, ld_in)
    X[:, :b.F] = torch.from_numpy(src).cuda()
    store = torch.full((rows * ld_out + out_off + 8,), SENTINEL, device="cuda")
    Y = store[out_off:out_off + rows * ld_out].view(rows, ld_out)
    (K.bspmm_run_transposed if transposed else K.bspmm_run)(plan.handle, X, Y, ld_in, ld_out)
    torch.cuda.synchronize()
    assert bool((store[:out_off] == SENTINEL).all()) and bool((store[out_off + rows * ld_out:] == SENTINEL).all())
    assert bool((Y[:, b.F:] == SENTINEL).all())
    return Y[:, :b.F].cpu().numpy()


def _check(got, ref, scale, off, length):
    owned = np.zeros(got.shape[0], dtype=bool)
    for o, n in zip(off, length):
        owned[int(o):int(o) + int(n)] = True
    assert np.all(got[~owned] == SENTINEL)
    err = np.abs(got.astype(np.float64) - ref)[owned]
    assert not np.any(~(err <= 1e-5 * scale[owned])), "beyond 1e-5*S"


@pytest.mark.parametrize("F", [1, 2, 3, 5, 50, 63, 65, 100, 127, 255, 257, 301])
def test_every_width_both_directions(oracle, F):
    import torch
    b = W.random_general(900 + F, F=F, shapes=SHAPES, shuffle_blocks=True)
    plan = K.Plan(b)
    for transposed in (False, True):
        got = _run(torch, plan, b, transposed, 0, 0, 0, 0)
        ref, S = (oracle.transposed_batch if transposed else oracle.forward_batch)(b)
        _check(got, ref, S, b.b_row_off if transposed else b.c_row_off, b.cols if transposed else b.rows)


@pytest.mark.parametrize("F", [1, 3, 17, 50, 127, 301])
def test_lane_groups_share_long_rows(oracle, F):
    """Around the line from which a row counts as long (sixteen entries on average), around one and two lane
    groups per row, with and without room for the partial sums, an empty row and one that holds everything,
    rows gathered from memory."""
    import torch
    shapes = [(m, k, z) for m in (1, 2, 3, 9, 10, 19, 37, 128, 129) for k, z in ((1, 16 * m), (3, 17 * m), (90, 40 * m))]
    b = W.random_general(31 + F, F=F, shapes=shapes + [(2, 6000, 900), (1, 6000, 33)], with_dY=False)
    skew = W.random_general(32 + F, F=F, shapes=[(4, 150, 660)], with_dY=False)
    skew.rpt[:] = [0, 0, 659, 660, 660]
    for b in (b, skew):
        plan = K.Plan(b)
        got = _run(torch, plan, b, False, 0, 0, 0, 0)
        ref, S = oracle.forward_batch(b)
        _check(got, ref, S, b.c_row_off, b.rows)


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("F", [1, 3, 12, 17, 50, 100, 127, 300])
def test_long_rows_on_and_off_16_bytes(oracle, F, extra):
    """Around the lines at which rows are shared by lane groups or take a lane per float: 16, 64 and 100 entries on
    average, rows whose floats are half of the lanes and one row more, staged and in row blocks; widths that are a
    multiple of four floats with rows on 16 bytes and, one float further apart, off them."""
    import torch
    half = min(max(1, 128 // F), 20)
    shapes = [(m, k, z) for m in sorted({1, 2, half, half + 1, 2 * half + 1}) for k in (2, 90)
              for z in (16 * m, 16 * m + 1, 64 * m - 1, 64 * m, 100 * m)] + [(1, 90, 1500)]
    blocks = [(1, 6000, 900), (half, 6000, 64 * half), (half + 1, 6000, 65 * (half + 1)), (2, 6000, 33)]
    b = W.random_general(51 + F, F=F, shapes=shapes + blocks)
    plan = K.Plan(b)
    info = plan.info()
    assert info.items_in_bin[0][K.BIN_GENERIC] > 0 and info.items_in_bin[0][K.BIN_WORKGROUP] > len(shapes) // 2
    for transposed in (False, True):
        got = _run(torch, plan, b, transposed, 0, 0, extra, extra)
        ref, S = (oracle.transposed_batch if transposed else oracle.forward_batch)(b)
        _check(got, ref, S, b.b_row_off if transposed else b.c_row_off, b.cols if transposed else b.rows)


@pytest.mark.parametrize("F", [1, 3, 50, 127])
def test_operations_without_columns_read_nothing(F):
    """No operation has columns, so there is no dense input at all, wherever the (empty) blocks start."""
    import torch
    rows, zero = np.array([5, 300], dtype=np.int32), np.zeros(2, dtype=np.int64)
    rpt = torch.zeros(307, dtype=torch.int32, device="cuda")
    hb = K.HostBatch(rows, zero, zero, [0, 6], zero, [1, 2], [0, 5], rpt)
    ws = torch.empty(K.bspmm_workspace_bytes(hb, F), dtype=torch.uint8, device="cuda")
    plan = K.bspmm_create(hb, F, None, ws, ws.numel())
    C = torch.full((305, F), SENTINEL, device="cuda")
    K.bspmm_run(plan, None, C, F, F)
    torch.cuda.synchronize()
    assert not bool(C.any())
    K.bspmm_destroy(plan)


def test_leading_dimension_that_is_the_width_in_its_low_32_bits():
    """Two rows 16 GiB apart are not a packed matrix (17 floats wide: 2^32 + 17 floats from row to row)."""
    import torch
    F, ld = 17, (1 << 32) + 17
    store = torch.empty(ld + F, device="cuda")
    store[F:2 * F] = float("nan")                         # what a packed second row would be
    b = W.random_general(3, F, [(6, 2, 12)])
    for r in range(2):
        store[r * ld:r * ld + F] = torch.from_numpy(b.B[r]).cuda()
    plan = K.Plan(b)
    got, want = torch.empty((6, F), device="cuda"), torch.empty((6, F), device="cuda")
    K.bspmm_run(plan.handle, store, got, ld, F)
    plan.run(torch.from_numpy(b.B).cuda(), want)
    assert torch.equal(got, want)


@pytest.mark.parametrize("F", [48, 50, 61])
@pytest.mark.parametrize("in_off,out_off,in_extra,out_extra", [(1, 0, 0, 0), (2, 3, 0, 0), (0, 1, 0, 0), (0, 0, 1, 3),
                                                               (4, 0, 2, 0), (3, 1, 5, 2)])
def test_operands_off_16_bytes(oracle, F, in_off, out_off, in_extra, out_extra):
    import torch
    b = W.random_general(40 + F, F=F, shapes=SHAPES)
    plan = K.Plan(b)
    for transposed in (False, True):
        got = _run(torch, plan, b, transposed, in_off, out_off, in_extra, out_extra)
        ref, S = (oracle.transposed_batch if transposed else oracle.forward_batch)(b)
        _check(got, ref, S, b.b_row_off if transposed else b.c_row_off, b.cols if transposed else b.rows)


@pytest.mark.parametrize("F", [4, 8, 16, 32, 64, 128])
@pytest.mark.parametrize("in_off", [0, 1])
def test_small_operations_share_a_workgroup(oracle, F, in_off):
    """More small operations than the chip holds workgroups: four to a workgroup, one wavefront each (up to
    two passes of rows), next to those that are too large for it; the same table off 16 bytes."""
    import torch
    limit = 512 // F
    one = [(limit, 9, 60), (limit - 1, 40, 190), (1, 1, 1), (limit, 3, 0), (0, 0, 0), (limit + 1, 20, 70), (2, 5, 7),
           (3 * limit, 30, 129)]
    b = W.random_general(77 + F, F=F, shapes=one * 500)
    plan = K.Plan(b)
    assert plan.info().items_in_bin[0][K.BIN_WAVE] > 0
    for transposed in (False, True):
        got = _run(torch, plan, b, transposed, in_off, 0, 0, 0)
        ref, S = (oracle.transposed_batch if transposed else oracle.forward_batch)(b)
        _check(got, ref, S, b.b_row_off if transposed else b.c_row_off, b.cols if transposed else b.rows)


@pytest.mark.parametrize("F,flags", [(50, 0), (100, 0), (127, 0), (64, 0), (128, 0), (64, K.ACCUMULATE),
                                     (50, K.ACCUMULATE)])
@pytest.mark.parametrize("shapes", [SHAPES, [(30, 40, 85)] * 12, [(8, 9, 31)] * 4000])
def test_infinite_and_nan_inputs(oracle, F, flags, shapes):
    """Infinities stay infinities: entries that fill up the last trip of a row count as nothing, not as
    0 * inf (staged tiles, row blocks, long rows, small operations, summed sets)."""
    import torch
    b = W.random_general(5 + F, F=F, shapes=shapes)
    if flags & K.ACCUMULATE:                           # pairs of operations of one shape, summed
        for i in range(1, b.batch, 2):
            if b.rows[i] == b.rows[i - 1]:
                b.c_row_off[i] = b.c_row_off[i - 1]
    rng = np.random.default_rng(F)
    for x in (b.B, b.dY):
        x[rng.random(x.shape) < 0.03] = np.inf
        x[rng.random(x.shape) < 0.03] = -np.inf
        x[rng.random(x.shape) < 0.002] = np.nan
    plan = K.Plan(b, F, K.make_options(flags=flags))
    got = torch.zeros((b.n_c_rows, F), device="cuda")
    plan.run(torch.from_numpy(b.B).cuda(), got)
    got = got.cpu().numpy()
    ref = np.zeros((b.n_c_rows, F))
    with np.errstate(invalid="ignore"):
        for i in range(b.batch):
            rpt = b.rpt[b.rpt_off[i]:b.rpt_off[i] + b.rows[i] + 1]
            at = slice(b.nz_off[i], b.nz_off[i] + b.nnz[i])
            row = np.repeat(np.arange(b.rows[i]), np.diff(rpt))
            np.add.at(ref, b.c_row_off[i] + row,
                      b.values[at, None].astype(np.float64) * b.B[b.b_row_off[i] + b.colids[at]])
    assert np.isinf(ref).any() and np.isnan(ref).any()
    finite = np.isfinite(ref)
    np.testing.assert_array_equal(got[~finite], ref[~finite].astype(np.float32))
    assert np.isfinite(got[finite]).all()
