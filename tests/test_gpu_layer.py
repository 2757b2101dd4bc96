"""The gather-first layer kernel (bspmm_layer_kernel) at the sizes where it can go wrong: last blocks that
are not full, columns that no tile divides, every number of channels, sums over more channels than one
launch holds, rows with more entries than a block has slots, numbers that the three-way bf16 split does not
hold and those it holds only scaled, strided operands, replays of a captured run.  Tolerances as in test_gpu_gcn."""
import dataclasses

import numpy as np
import pytest

from paper_1903_11409_amd import bspmm as K
from paper_1903_11409_amd import workloads as W
from test_gpu_gcn import SENTINEL, _assert_close, _channel, _layer, _owned, _tol, torch_cuda  # noqa: F401
from test_schedule_cpu import _of_degree

pytestmark = pytest.mark.gpu


def _reference(oracle, b, X, Ws, biases):
    Y = T = None
    for c in range(len(Ws)):
        Y, T = oracle.gcn_channel(_channel(b, c, len(Ws)), X, Ws[c], biases[c], Y, T)
    return Y, T


def _plan(b, n_x, chans, **kw):
    return K.Plan(b, options=K.make_options(flags=K.ACCUMULATE if chans > 1 else 0, front_features=n_x, **kw))


def _device(torch, X, Ws, biases):
    return (torch.from_numpy(X).cuda(), torch.from_numpy(np.concatenate(Ws, axis=0)).cuda(),
            torch.from_numpy(np.stack(biases)).cuda())


def _batch(graphs, F, chans):
    if chans == 1:
        return W.config2_molecule(seed=40 + graphs, graphs=graphs, F=F)
    return W.config3_multichannel(seed=40 + graphs, graphs=graphs, F=F, channels=chans, accumulate=True)


@pytest.mark.parametrize("graphs,chans,n_x,F", [
    # one channel: blocks of one operation from its own arrays (few graphs), and blocks across graphs; one, two
    # and four 16-row blocks a trip; K = channels n_x from one step of 32 to sixteen, off steps
    # (16, 48, 80, 112), and past what one launch adds up (5 and 8 channels of 128)
    (700, 1, 16, 64), (700, 1, 32, 128), (90, 1, 64, 128), (700, 1, 64, 256), (90, 1, 128, 16), (90, 1, 128, 144),
    (90, 2, 16, 48), (500, 2, 32, 64), (90, 2, 64, 80), (90, 2, 128, 128), (90, 3, 16, 128), (90, 3, 32, 96),
    (90, 3, 64, 128), (90, 3, 128, 64), (90, 4, 16, 16), (90, 4, 64, 128), (300, 4, 128, 128), (90, 5, 16, 128),
    (60, 5, 128, 64), (90, 7, 16, 80), (60, 7, 64, 128), (60, 8, 32, 128), (60, 8, 64, 64), (40, 8, 128, 128)])
def test_every_shape_of_a_workgroup(torch_cuda, oracle, graphs, chans, n_x, F):  # noqa: F811
    torch = torch_cuda
    b = _batch(graphs, F, chans)
    X, Ws, biases = _layer(b, n_x, 7, channels=chans)
    Xd, Wd, bd = _device(torch, X, Ws, biases)
    ref, T = _reference(oracle, b, X, Ws, biases)
    owned = _owned(b.c_row_off, b.rows, b.n_c_rows)
    for kw in ({}, {"compute_units": 8}):          # a block or two to a workgroup, and many
        print(f"layer {graphs} graphs, {chans} channels, n_x {n_x}, F {F} {kw}", flush=True)
        plan = _plan(b, n_x, chans, **kw)
        Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
        plan.run_gcn(Xd, Wd, bd, Yd)
        plan_again = torch.empty_like(Yd)
        plan.run_gcn(Xd, Wd, bd, plan_again)
        base = torch.rand_like(Yd)
        onto = base.clone()
        plan.run_gcn(Xd, Wd, bd, onto, accumulate=True)
        torch.cuda.synchronize()
        got = Yd.cpu().numpy()
        _assert_close(got, ref, T, owned, max(1e-5, chans * (n_x + 10) * 2.0 ** -23), "layer")
        assert torch.equal(Yd[torch.from_numpy(owned).cuda()], plan_again[torch.from_numpy(owned).cuda()])
        # roundings of K products and a few entries, independent of each other
        err = np.linalg.norm(got[owned] - ref[owned]) / np.linalg.norm(ref[owned])
        assert err <= 2.0 ** -24 * np.sqrt(chans * n_x + 16), err
        added = onto.cpu().numpy().astype(np.float64) - base.cpu().numpy()
        assert np.all(np.abs(added - ref)[owned] <= 1e-5 * (T + 1)[owned])
        assert np.array_equal(added[~owned], np.zeros_like(added[~owned]))


@pytest.mark.parametrize("chans,cus", [(1, 1), (1, 0), (3, 1)])
@pytest.mark.parametrize("n_x", [16, 64, 128])
def test_rows_with_more_entries_than_slots(torch_cuda, oracle, chans, cus, n_x):  # noqa: F811
    """A star: one row names every node, all others name one; a block's entries do not fit its slots."""
    torch = torch_cuda
    rng = np.random.default_rng(3)
    n, graphs, F = 300, 6, 64
    ops, block = [], []
    for g in range(graphs):
        for c in range(chans):
            counts = np.ones(n, dtype=np.int32)
            counts[(7 * g + c) % n] = n - 1
            rpt = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
            ci = rng.integers(0, n, int(rpt[-1])).astype(np.int32)
            ops.append((n, n, rpt, ci, rng.uniform(-1, 1, int(rpt[-1])).astype(np.float32)))
            block.append(g)
    b = W.assemble("stars", F, ops, block, [n] * graphs, rng, n_graphs=graphs, c_block_of_op=block)
    X, Ws, biases = _layer(b, n_x, 2, channels=chans)
    Xd, Wd, bd = _device(torch, X, Ws, biases)
    plan = _plan(b, n_x, chans, compute_units=cus)
    Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
    plan.run_gcn(Xd, Wd, bd, Yd)
    torch.cuda.synchronize()
    ref, T = _reference(oracle, b, X, Ws, biases)
    _assert_close(Yd.cpu().numpy(), ref, T, _owned(b.c_row_off, b.rows, b.n_c_rows),
                  max(1e-5, chans * (n_x + n) * 2.0 ** -23), "stars")


@pytest.mark.parametrize("chans,n_x,F", [(1, 16, 64), (1, 64, 128), (2, 32, 128), (1, 128, 64), (4, 64, 128),
                                         (5, 128, 128), (6, 16, 128), (8, 128, 128)])
@pytest.mark.parametrize("per_row,heavy,cus", [(8, None, 4), (20, None, 4), (100, None, 2), (3, 70, 4), (7, None, 0)])
def test_many_entries_per_row(torch_cuda, oracle, chans, n_x, F, per_row, heavy, cus):  # noqa: F811
    """Blocks inside their slots, past them (rows of more entries than a lane group requests at once, and of
    fewer) and graphs of many entries in a launch of their own, beside graphs of few."""
    torch = torch_cuda
    b = _of_degree(60, chans, per_row, heavy, F=F)
    X, Ws, biases = _layer(b, n_x, 8, channels=chans)
    plan = _plan(b, n_x, chans, compute_units=cus)
    ops = _device(torch, X, Ws, biases)
    Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
    plan.run_gcn(*ops, Yd)
    onto = torch.ones_like(Yd)
    plan.run_gcn(*ops, onto, accumulate=True)
    torch.cuda.synchronize()
    ref, T = _reference(oracle, b, X, Ws, biases)
    tol = max(1e-5, (chans * n_x + (heavy or per_row) + 10) * 2.0 ** -23)
    _assert_close(Yd.cpu().numpy(), ref, T, _owned(b.c_row_off, b.rows, b.n_c_rows), tol, "many entries")
    assert np.all(np.abs(onto.cpu().numpy().astype(np.float64) - 1 - ref) <= tol * (T + 1))


@pytest.mark.parametrize("chans,n_x,F,cus", [(1, 64, 128, 8), (1, 64, 128, 0), (4, 64, 128, 8), (2, 16, 64, 0)])
def test_numbers_that_do_not_split(torch_cuda, oracle, chans, n_x, F, cus):  # noqa: F811
    """Infinities, NaN and numbers near the end of the range reach the rows that name them and no others;
    operands as small as 1e-36 keep their bits."""
    torch = torch_cuda
    b = _batch(80, F, chans)
    X, Ws, biases = _layer(b, n_x, 5, channels=chans)
    owned = _owned(b.c_row_off, b.rows, b.n_c_rows)
    plan = _plan(b, n_x, chans, compute_units=cus)

    def run(X, Ws, biases):
        Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
        plan.run_gcn(*_device(torch, X, Ws, biases), Yd)
        torch.cuda.synchronize()
        return Yd.cpu().numpy().astype(np.float64)

    def channels_of(bad_row):        # which owned output rows name that row of X
        hit = np.zeros(b.n_c_rows, dtype=bool)
        for i in range(b.batch):
            rpt, ci, _ = b.op_csr(i)
            rows = np.repeat(np.arange(len(rpt) - 1), np.diff(rpt))
            hit[int(b.c_row_off[i]) + rows[ci + int(b.b_row_off[i]) == bad_row]] = True
        return hit

    ref, T = _reference(oracle, b, X, Ws, biases)
    tol = max(1e-5, chans * (n_x + 10) * 2.0 ** -23)
    for bad in (np.inf, -np.inf, np.nan):
        X2 = X.copy()
        X2[37, n_x // 2] = bad
        got, hit = run(X2, Ws, biases), channels_of(37)
        assert not np.any(np.isfinite(got[hit])), bad
        _assert_close(np.where(hit[:, None], ref, got), ref, T, owned, tol, f"rows beside {bad}")
    # a weight that is not finite: its column, in rows with entries in its channel
    Ws2 = [w.copy() for w in Ws]
    Ws2[-1][3, 5] = np.inf
    got = run(X, Ws2, biases)
    last = _channel(b, chans - 1, chans)
    named = np.zeros(b.n_c_rows, dtype=bool)
    for i in range(last.batch):
        named[int(last.c_row_off[i]):][:int(last.rows[i])] |= np.diff(last.op_csr(i)[0]) > 0
    touched = np.zeros((b.n_c_rows, F), dtype=bool)
    touched[named, 5] = True
    assert not np.any(np.isfinite(got[touched]))
    _assert_close(np.where(touched, ref, got), ref, T, owned, tol, "columns beside an infinite weight")
    # the largest finite numbers: bf16 rounds them to infinity
    X2 = X.copy()
    X2[37] = 3.4e38
    Ws2 = [w * np.float32(1e-3) for w in Ws]
    ref2, T2 = _reference(oracle, b, X2, Ws2, biases)
    small = np.abs(ref2).max(axis=1) < 1e38       # (the products of the gather stay in range there)
    got = run(X2, Ws2, biases)
    _assert_close(np.where(small[:, None], got, ref2), ref2, T2, owned, tol, "large numbers")
    for scale in (1e-12, 1e-30, 1e-36):
        X2, none = X * np.float32(scale), [np.zeros_like(v) for v in biases]
        ref2, T2 = _reference(oracle, b, X2, Ws, none)
        _assert_close(run(X2, Ws, none), ref2, T2, owned, tol, f"scale {scale}")


@pytest.mark.parametrize("chans,n_x,F,cus", [(1, 64, 128, 8), (1, 64, 128, 0), (4, 64, 128, 8), (2, 16, 64, 0)])
def test_tiny_graphs_beside_ordinary_ones(torch_cuda, oracle, chans, n_x, F, cus):  # noqa: F811
    """Rows of 1e-36, or a column of weights, beside ordinary ones in the same block keep their bits too:
    the bound is each element's own sum of magnitudes."""
    torch = torch_cuda
    b = _batch(80, F, chans)
    X, Ws, _ = _layer(b, n_x, 6, channels=chans)
    none = [np.zeros(F, dtype=np.float32)] * chans
    X2, Ws2 = X.copy(), [w.copy() for w in Ws]
    for i in range(0, b.batch, 3 * chans):
        X2[int(b.b_row_off[i]):int(b.b_row_off[i]) + int(b.cols[i])] *= np.float32(1e-36)
    for w in Ws2:
        w[:, 5] *= np.float32(1e-36)
    owned = _owned(b.c_row_off, b.rows, b.n_c_rows)
    plan = _plan(b, n_x, chans, compute_units=cus)
    for x, w in ((X2, Ws), (X, Ws2)):
        Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
        plan.run_gcn(*_device(torch, x, w, none), Yd)
        torch.cuda.synchronize()
        ref, T = _reference(oracle, b, x, w, none)
        # (products of 1e-36 that come out subnormal: half of the smallest number each)
        _assert_close(Yd.cpu().numpy(), ref, T + 1e-38, owned, max(1e-5, chans * (n_x + 10) * 2.0 ** -23), "tiny")


def _scaled(b, n_x, chans, sx, sw, sa):
    """Operands of the layer and their values of A, scaled; the bias as large as the products."""
    X, Ws, biases = _layer(b, n_x, 11, channels=chans)
    f = np.float32
    return (dataclasses.replace(b, values=b.values * f(sa)), X * f(sx), [w * f(sw) for w in Ws],
            [v * f(float(sx) * sw) for v in biases])


# every way the blocks are made again: from an operation's own arrays or across graphs, one and two 16-column
# blocks per wavefront, one to four 16-row blocks, four and eight wavefronts, two launches
WAYS = [(1, 64, 128, 0), (1, 64, 128, 8), (1, 32, 128, 0), (1, 32, 128, 8), (1, 16, 64, 8), (2, 16, 64, 8),
        (4, 64, 128, 8), (5, 32, 128, 8), (8, 64, 128, 8), (8, 128, 64, 8)]


@pytest.mark.parametrize("chans,n_x,F,cus", WAYS)
def test_sums_that_only_the_layers_own_order_holds(torch_cuda, oracle, chans, n_x, F, cus):  # noqa: F811
    """A X is past the largest number, X W and A (X W + bias) are not; also onto what Y holds."""
    torch = torch_cuda
    b, X, Ws, biases = _scaled(_batch(80, F, chans), n_x, chans, 1e38, 1e-10, 1e3)
    ref, T = _reference(oracle, b, X, Ws, biases)
    owned = _owned(b.c_row_off, b.rows, b.n_c_rows)
    tol = max(1e-5, chans * (n_x + 10) * 2.0 ** -23)
    plan = _plan(b, n_x, chans, compute_units=cus)
    ops = _device(torch, X, Ws, biases)
    Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
    plan.run_gcn(*ops, Yd)
    onto = torch.full_like(Yd, 2.0 ** 100)
    plan.run_gcn(*ops, onto, accumulate=True)
    torch.cuda.synchronize()
    _assert_close(Yd.cpu().numpy(), ref, T, owned, tol, "order of the sums")
    added = onto.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(added - 2.0 ** 100 - ref)[owned] <= tol * (T + 2.0 ** 100)[owned])
    assert np.all(added[~owned] == 2.0 ** 100)


# X, W, A: small operands beside large ones, the result ordinary or tiny, inside the weights that the split
# takes (2^16) and past them, subnormal ones, and A X below the smallest number
SCALES = [(1e-36, 1e20, 1), (1e20, 1e-36, 1), (1e-37, 1e30, 1), (1e30, 1e-37, 1), (1e-36, 3e4, 1), (1e8, 1e-36, 1),
          (1e-37, 1, 1), (1, 1e-37, 1), (1e-41, 3e4, 1e-2), (1e8, 1e-41, 1e-2), (1e-30, 1e30, 1e-30),
          (1e-30, 3e4, 1e-10), (1, 3e4, 1e-36), (1e14, 3e4, 1e-3), (1e10, 1e5, 1e3)]


@pytest.mark.parametrize("chans,n_x,F,cus", WAYS)
def test_small_operands_beside_large_ones(torch_cuda, oracle, chans, n_x, F, cus):  # noqa: F811
    """No bits are lost at the lower end of the range whatever the other operand is, alone or in a block of
    ordinary rows, and onto what Y holds: the bound is each element's own sum of magnitudes, and half of the
    smallest number for every product that comes out subnormal."""
    torch = torch_cuda
    batch = _batch(80, F, chans)
    owned = _owned(batch.c_row_off, batch.rows, batch.n_c_rows)
    tol = max(1e-5, chans * (n_x + 10) * 2.0 ** -23)
    for sx, sw, sa in SCALES:
        for beside in (False, True):
            b, X, Ws, biases = _scaled(batch, n_x, chans, sx, sw, sa)
            if beside:                     # every third graph; the others are ordinary
                ordinary = np.ones(b.n_b_rows, dtype=bool)
                for i in range(0, b.batch, 3 * chans):
                    ordinary[int(b.b_row_off[i]):int(b.b_row_off[i]) + int(b.cols[i])] = False
                X[ordinary] /= np.float32(sx)
                biases = [np.zeros_like(v) for v in biases]
            ref, T = _reference(oracle, b, X, Ws, biases)
            plan = _plan(b, n_x, chans, compute_units=cus)
            ops = _device(torch, X, Ws, biases)
            Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
            plan.run_gcn(*ops, Yd)
            onto = torch.zeros_like(Yd)
            plan.run_gcn(*ops, onto, accumulate=True)
            torch.cuda.synchronize()
            floor = 2.0 ** -149 * (chans * n_x + 16) / tol
            for got in (Yd, onto):
                _assert_close(got.cpu().numpy(), ref, T + floor, owned if got is Yd else np.ones_like(owned), tol,
                              f"X {sx} W {sw} A {sa}")


@pytest.mark.parametrize("chans,n_x,F,cus", WAYS)
def test_one_weight_that_is_no_number(torch_cuda, oracle, chans, n_x, F, cus):  # noqa: F811
    """It reaches its column in the rows with entries in its channel, and every block is made again."""
    torch = torch_cuda
    b = _batch(80, F, chans)
    X, Ws, biases = _layer(b, n_x, 12, channels=chans)
    ref, T = _reference(oracle, b, X, Ws, biases)
    Ws[-1][n_x - 1, 37] = np.nan
    plan = _plan(b, n_x, chans, compute_units=cus)
    Yd = torch.full((b.n_c_rows, F), SENTINEL, dtype=torch.float32, device="cuda")
    plan.run_gcn(*_device(torch, X, Ws, biases), Yd)
    torch.cuda.synchronize()
    got = Yd.cpu().numpy()
    last = _channel(b, chans - 1, chans)
    touched = np.zeros((b.n_c_rows, F), dtype=bool)
    for i in range(last.batch):
        touched[int(last.c_row_off[i]):][:int(last.rows[i]), 37] |= np.diff(last.op_csr(i)[0]) > 0
    assert np.all(np.isnan(got[touched]))
    _assert_close(np.where(touched, ref, got), ref, T, _owned(b.c_row_off, b.rows, b.n_c_rows),
                  max(1e-5, chans * (n_x + 10) * 2.0 ** -23), "beside a NaN")


def test_static_workspace_holds_layers_without_the_gather_first_arrays(torch_cuda, oracle):  # noqa: F811
    """Many entries: the static array holds the plan, but not with the layer's arrays beside the transposed CSR."""
    torch = torch_cuda
    b, n_x = _of_degree(800, 1, 30), 128
    options = K.make_options(front_features=n_x)
    dry = [K.dry_plan(b, b.F, front_features=n_x, flags=flags) for flags in (0, K.ONE_FRONT_LAUNCH)]
    size = [int(K.bspmm_plan_info(h).workspace_bytes) for h in dry]
    for h in dry:
        K.bspmm_destroy(h)
    assert size[0] > K.STATIC_WORKSPACE_BYTES >= size[1], size
    arrays = [torch.from_numpy(a).cuda() for a in (b.rpt, b.colids, b.values)]
    plan = K.bspmm_create_static(K.HostBatch(b.rows, b.cols, b.nnz, b.rpt_off, b.nz_off, b.b_row_off, b.c_row_off,
                                             *arrays), b.F, options)
    X, Ws, biases = _layer(b, n_x, 3)
    Xd, Wd, bd = _device(torch, X, Ws, biases)
    Yd = torch.full((b.n_c_rows, b.F), SENTINEL, dtype=torch.float32, device="cuda")
    K.bspmm_run_gcn(plan, Xd, n_x, Wd, b.F, bd, Yd, b.F)
    torch.cuda.synchronize()
    ref, T = _reference(oracle, b, X, Ws, biases)
    _assert_close(Yd.cpu().numpy(), ref, T, _owned(b.c_row_off, b.rows, b.n_c_rows), 1e-5, "static")
    K.bspmm_destroy(plan)


def test_resources_of_the_layer_kernel_are_those_of_the_variant_that_runs(torch_cuda):  # noqa: F811
    """Four channels of 64 at F = 128: workgroups of eight wavefronts, nothing spilled."""
    b = _batch(2048, 128, 4)
    info = _plan(b, 64, 4).info()
    kernel = K.bspmm_kernel_info(8, int(info.front_stream[2]))
    assert (kernel.threads, kernel.scratch_bytes) == (512, 0) and 64 < kernel.vgprs <= 128
    assert info.front_stream[1] <= kernel.workgroups_per_cu * kernel.compute_units


def test_identity_weights_give_the_plain_product(torch_cuda):  # noqa: F811
    """W = I, bias = 0: a sum of three bf16 numbers is the fp32 number they were made from."""
    torch = torch_cuda
    b = W.config2_molecule(graphs=300, F=64)
    plan = _plan(b, 64, 1)
    Xd = torch.from_numpy(b.B).cuda()
    Y1, Y2 = (torch.empty((b.n_c_rows, 64), dtype=torch.float32, device="cuda") for _ in range(2))
    plan.run_gcn(Xd, torch.eye(64, device="cuda"), torch.zeros(64, device="cuda"), Y1)
    plan.run(Xd, Y2)
    torch.cuda.synchronize()
    assert torch.equal(Y1, Y2)


@pytest.mark.parametrize("graphs", [100, 900])
def test_strides_scattered_blocks_and_a_wide_weight_matrix(torch_cuda, oracle, graphs):  # noqa: F811
    """Strided X, W and Y; output blocks in another order than the input's, with gaps; a weight matrix whose
    rows are too far apart for 32-bit offsets takes the one-launch kernel."""
    torch = torch_cuda
    b = W.config2_molecule(seed=9, graphs=graphs, F=64)
    n_x, order = 16, np.random.default_rng(1).permutation(graphs)
    c_off = np.zeros(graphs, dtype=np.int64)
    c_off[order] = np.cumsum(np.concatenate([[3], b.rows[order][:-1] + 2]))
    b = dataclasses.replace(b, c_row_off=c_off, n_c_rows=int((c_off + b.rows).max()) + 5)
    X, Ws, biases = _layer(b, n_x, 4)
    ref, T = oracle.gcn_channel(b, X, Ws[0], biases[0])
    plan = _plan(b, n_x, 1)
    Xd = torch.zeros((b.n_b_rows, n_x + 8), device="cuda")
    Xd[:, :n_x] = torch.from_numpy(X).cuda()
    for ldw in (68, 1 << 20):
        Wd = torch.zeros((n_x, ldw), device="cuda")
        Wd[:, :64] = torch.from_numpy(Ws[0]).cuda()
        Yd = torch.full((b.n_c_rows, 76), SENTINEL, dtype=torch.float32, device="cuda")
        K.bspmm_run_gcn(plan.handle, Xd, n_x + 8, Wd, ldw, torch.from_numpy(biases[0]).cuda(), Yd, 76)
        torch.cuda.synchronize()
        _assert_close(Yd[:, :64].cpu().numpy(), ref, T, _owned(b.c_row_off, b.rows, b.n_c_rows), _tol(b, n_x), f"ldw {ldw}")
        assert torch.all(Yd[:, 64:] == SENTINEL)


@pytest.mark.parametrize("built", [False, True])
def test_replays_of_a_captured_layer(torch_cuda, oracle, built):  # noqa: F811
    """A first run inside a capture records the kernel that writes the blocks' arrays too; replays, with
    eager runs between them, give what an eager run gives and what the oracle does."""
    torch = torch_cuda
    b = _batch(200, 128, 4)
    X, Ws, biases = _layer(b, 64, 5, channels=4)
    Xd, Wd, bd = _device(torch, X, Ws, biases)
    plan = K.Plan(b, options=K.make_options(flags=K.ACCUMULATE | (K.BUILD_TRANSPOSE if built else 0), front_features=64))
    Y = torch.zeros((b.n_c_rows, 128), device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.run_gcn(Xd, Wd, bd, Y)
    other = torch.empty_like(Y)
    for i in range(3):
        Xd.copy_(torch.from_numpy(X * (i + 1)).cuda())
        Y.zero_()
        g.replay()
        torch.cuda.synchronize()
        plan.run_gcn(Xd, Wd, bd, other)
        torch.cuda.synchronize()
        owned = _owned(b.c_row_off, b.rows, b.n_c_rows)
        assert torch.equal(Y[owned], other[owned])
        ref, T = _reference(oracle, b, X * np.float32(i + 1), Ws, biases)
        got = Y.cpu().numpy()
        assert np.all(got[~owned] == 0)
        got[~owned] = SENTINEL
        _assert_close(got, ref, T, owned, max(1e-5, 4 * (64 + 10) * 2.0 ** -23), f"replay {i}")
