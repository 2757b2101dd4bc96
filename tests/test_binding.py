"""The binding's own decisions: leading dimensions and streams of the native run calls, and which
outputs of the autograd wrapper have to be cleared first."""
import numpy as np
import pytest

from paper_1903_11409_amd import bspmm as K
from paper_1903_11409_amd import workloads as W


@pytest.mark.parametrize("blocks", [[], [(0, 4)], [(4, 3), (0, 4)], [(1, 4)], [(0, 4), (5, 2)], [(0, 4), (4, 0), (4, 1)],
                                    [(0, 4), (0, 4), (4, 5)], [(7, 2), (0, 3), (3, 3)]])
def test_rows_covered_from_the_first_on(blocks):
    off = np.array([b[0] for b in blocks], dtype=np.int64)
    length = np.array([b[1] for b in blocks], dtype=np.int32)
    hit = np.zeros(16, dtype=bool)
    for o, n in blocks:
        hit[o:o + n] = True
    zero = np.zeros(len(off), dtype=np.int64)
    hb = K.HostBatch(length, length, zero, zero, zero, off, off)
    for flags in (K.DRY_RUN | K.ACCUMULATE, K.DRY_RUN):
        try:
            plan = K.bspmm_create(hb, 8, K.make_options(flags=flags))
        except K.BspmmError as e:       # blocks that overlap without being the same belong to no batch
            assert e.code == K.EOVERLAP
            continue
        assert K.native().covered_rows(plan, False) == K.native().covered_rows(plan, True) == int(np.argmin(hit))
        K.bspmm_destroy(plan)


def test_native_calls_check_their_arguments():
    n = K.native()
    for call in (lambda: n.run(None, None, None, 1, 1, 0), lambda: n.run_transposed(None, None, None, 1, 1, 0),
                 lambda: n.run_gcn(None, None, None, None, None, 1, 1, 1, False, 0)):
        with pytest.raises(K.BspmmError) as e:
            call()
        assert e.value.code == K.EINVAL
    with pytest.raises(TypeError):
        n.run(None, None)
    with pytest.raises(TypeError):
        n.run(None, None, None, "x", 1, 0)


WAIT = r"""
#include "staging.hpp"
#include <cstdio>
int main()
{
    using bspmm::wait_until;
    int asked = 0;
    auto state = [&](hipError_t last, int after) { return [&asked, last, after] { return ++asked > after ? last : hipErrorNotReady; }; };
    auto never = [] { return false; };
    auto now = [] { return true; };
    if (wait_until(now, state(hipErrorUnknown, 0)) != hipSuccess || asked != 0) return 1;     // not asked at once
    if (wait_until(never, state(hipErrorLaunchFailure, 2)) != hipErrorLaunchFailure || asked != 3) return 2;
    asked = 0;
    if (wait_until(never, state(hipSuccess, 1)) != hipErrorUnknown) return 3;   // the stream is through, the copy is not
    asked = 0;
    if (wait_until([&] { return asked > 4; }, state(hipSuccess, 4)) != hipSuccess) return 4;    // done while it was asked
    std::puts("ok");
}
"""


def test_wait_for_the_tables_ends_with_the_error_of_the_stream(tmp_path):
    """A copy that never runs is an error of the call that waits for it, not a wait without end."""
    import os
    import subprocess
    from paper_1903_11409_amd import build
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(WAIT)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I" + build.CSRC,
                    "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), str(src), "-o",
                    str(exe), "-pthread"], check=True, timeout=120)
    assert subprocess.run([str(exe)], capture_output=True, timeout=30, text=True).stdout == "ok\n"


def test_library_is_built_without_pytorch():
    """A user of the C ABI has neither PyTorch nor numpy; the compiler is left out here."""
    import subprocess
    import sys
    from paper_1903_11409_amd import build
    code = ("import importlib.util, os, sys\n"
            "sys.modules['torch'] = sys.modules['numpy'] = None\n"
            "os.environ['HIPCC'] = '/bin/true'\n"
            "spec = importlib.util.spec_from_file_location('build', sys.argv[1])\n"
            "m = importlib.util.module_from_spec(spec)\n"
            "spec.loader.exec_module(m)\n"
            "print(m.build_library())\n")
    r = subprocess.run([sys.executable, "-c", code, build.__file__], capture_output=True, text=True, timeout=60)
    assert r.stdout.strip() == build.LIB, r.stderr


POOL = r"""
#include "staging.hpp"
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <vector>
// The runtime's part: freeing waits for the device, here for another thread that takes a block meanwhile.
static std::atomic<int> freeing{0}, taken{0};
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p)
{
    freeing = 1;
    for (int i = 0; i < 2000 && !taken; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    std::free(p);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus*) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}
namespace bspmm {
hipError_t launch_stage_copy(const void*, void*, size_t, uint32_t* done, uint32_t mark, int grid, hipStream_t)
{
    for (int i = 0; i < grid; ++i) done[i] = mark;
    return hipSuccess;
}
}
int main()
{
    using namespace bspmm;
    std::vector<StageBlock> blocks;
    for (size_t held = 0; held < kStagePoolMax; held += (size_t)256 << 10) blocks.push_back(stage_take(1));   // full
    if (!blocks.back().ptr) return 1;
    StagedCopy copy;
    for (StageBlock& b : blocks)
        if (stage_copy(b, nullptr, 16, nullptr, &copy) != hipSuccess) return 2;
    std::thread other([] {
        while (!freeing) std::this_thread::yield();
        if (stage_take(1).ptr) taken = 1;
    });
    const bool got = stage_take(kStageBlockMax).ptr != nullptr;      // makes room
    const bool meanwhile = taken;
    other.join();
    std::puts(got && meanwhile ? "ok" : "waited");
}
"""


def test_room_in_the_staging_pool_is_made_outside_its_lock(tmp_path):
    """Freeing pinned memory may wait for the device: other threads go on making plans meanwhile."""
    import os
    import subprocess
    from paper_1903_11409_amd import build
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(POOL)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I" + build.CSRC,
                    "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), str(src),
                    os.path.join(build.CSRC, "staging.cpp"), "-o", str(exe), "-pthread"], check=True, timeout=120)
    assert subprocess.run([str(exe)], capture_output=True, timeout=60, text=True).stdout == "ok\n"


@pytest.mark.gpu
@pytest.mark.parametrize("rows,ld", [(1, 64), (1, 72), (7, 64), (7, 68), (7, 65)])
@pytest.mark.parametrize("stream", ["current", "object", "handle"])
def test_leading_dimension_and_stream_of_a_plan_call(rows, ld, stream):
    import torch
    b = W.identity_batch(3, 64, [rows])
    plan = K.Plan(b, device="cuda:0")
    B = torch.zeros((rows, ld), device="cuda:0")
    B[:, :64] = torch.from_numpy(b.B)
    C = torch.full((rows, ld), -7.0, device="cuda:0")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        given = {"current": None, "object": side, "handle": side.cuda_stream}[stream]
        assert plan.run(B[:, :64], C[:, :64], given) is not None
        D = torch.empty_like(C)[:, :64]
        plan.run_transposed(C[:, :64], D, given)
    side.synchronize()
    assert torch.equal(C[:, :64].cpu(), torch.from_numpy(b.B)) and torch.equal(D.cpu(), torch.from_numpy(b.B))
    assert bool((C[:, 64:] == -7.0).all())
    with pytest.raises(K.BspmmError):
        K.bspmm_run(plan.handle, B, C, 63, ld)


@pytest.mark.gpu
@pytest.mark.parametrize("gap", [False, True])
def test_autograd_rows_of_no_operation_are_zero(gap):
    import torch
    from paper_1903_11409_amd.autograd import batched_spmm
    b = W.random_general(5, 12, [(9, 9, 30), (4, 4, 0), (11, 11, 25)], shuffle_blocks=gap)
    plan = K.Plan(b, device="cuda:0")
    rows = b.n_c_rows + (5 if gap else 0)
    torch.empty(1 << 16, device="cuda:0").fill_(float("nan"))     # what an uncleared output would show
    C = batched_spmm(plan, torch.from_numpy(b.B).cuda().requires_grad_(), rows)
    covered = np.zeros(rows, dtype=bool)
    for o, m in zip(b.c_row_off, b.rows):
        covered[int(o):int(o) + int(m)] = True
    got = C.detach().cpu().numpy()
    assert np.isfinite(got).all() and not got[~covered].any()


@pytest.mark.gpu
@pytest.mark.parametrize("made_on", ["current", "given"])
def test_plan_runs_on_another_stream_than_it_was_made_on(made_on):
    """No ordering between the streams by the caller: the tables (and the CSR arrays, from host memory)
    have arrived before the first launch, and the data loader may reuse its arrays at once."""
    import copy
    import torch
    from oracle import reference
    b = W.random_general(11, 48, [(40, 30, 200), (7, 7, 0), (90, 110, 500)])
    C0, S = reference.forward_batch(b)
    G0, SG = reference.transposed_batch(b)
    B, dY = torch.from_numpy(b.B).cuda(), torch.from_numpy(b.dY).cuda()
    side, busy = torch.cuda.Stream(), torch.randn((2048, 2048), device="cuda:0")
    torch.cuda.synchronize()
    for _ in range(4):
        loader = copy.deepcopy(b)
        with torch.cuda.stream(torch.cuda.current_stream() if made_on == "given" else side):
            with torch.cuda.stream(side):
                for _ in range(4):
                    busy @ busy            # the copy waits behind these
            plan = K.Plan(loader, device="cuda:0", stream=side if made_on == "given" else None)
            sizes = plan.rpt_len, plan.rpt_t_len, plan.nnz_total
            for a in (loader.rows, loader.cols, loader.nnz, loader.rpt, loader.colids, loader.values):
                a[:] = 0
            assert sizes == (plan.rpt_len, plan.rpt_t_len, plan.nnz_total)
            assert sizes == (int(b.rows.sum()) + 3, int(b.cols.sum()) + 3, int(b.nnz.sum()))
        other = torch.cuda.Stream()
        with torch.cuda.stream(other):
            C = plan.run(B, torch.zeros((b.n_c_rows, b.F), device="cuda:0"))
            G = plan.run_transposed(dY, torch.zeros((b.n_b_rows, b.F), device="cuda:0"))
        other.synchronize()
        # the bound of the other parity tests: 1e-5 of the sum of the products' magnitudes
        assert np.all(np.abs(C.cpu().numpy() - C0) <= 1e-5 * S)
        assert np.all(np.abs(G.cpu().numpy() - G0) <= 1e-5 * SG)
        torch.cuda.synchronize()


@pytest.mark.gpu
def test_plan_made_and_run_on_the_per_thread_streams_of_two_threads():
    """hipStreamPerThread is the same handle on both threads and two streams that nothing orders."""
    import threading
    import torch
    from oracle import reference
    per_thread = 2                         # (hipStream_t)2 in hip_runtime_api.h
    b = W.random_general(11, 48, [(40, 30, 200), (7, 7, 0), (90, 110, 500)])
    C0, S = reference.forward_batch(b)
    arrays = [torch.from_numpy(a).cuda() for a in (b.rpt, b.colids, b.values)]
    hb = K.HostBatch(b.rows, b.cols, b.nnz, b.rpt_off, b.nz_off, b.b_row_off, b.c_row_off, *arrays)
    need = K.bspmm_workspace_bytes(hb, b.F)
    ws, busy = torch.zeros(need, dtype=torch.uint8, device="cuda"), torch.ones(1 << 28, device="cuda")
    B, C = torch.from_numpy(b.B).cuda(), torch.full((b.n_c_rows, b.F), -7.0, device="cuda")
    torch.cuda.synchronize()
    made = []

    def make():
        with torch.cuda.stream(torch.cuda.ExternalStream(per_thread)):
            for _ in range(60):
                busy.mul_(1.0)             # the copy waits behind these
        made.append(K.bspmm_create(hb, b.F, None, ws, need, per_thread))

    t = threading.Thread(target=make)
    t.start()
    t.join()
    K.bspmm_run(made[0], B, C, b.F, b.F, per_thread)
    torch.cuda.synchronize()
    assert np.all(np.abs(C.cpu().numpy() - C0) <= 1e-5 * S)
    K.bspmm_destroy(made[0])


@pytest.mark.gpu
def test_plan_of_large_tables_runs_on_another_stream_than_it_was_made_on():
    """Tables beyond a staging block go over from pageable memory; a run on a stream that nothing orders
    behind that copy waits for it too."""
    import torch
    n, F = 140_000, 4                      # 64 bytes an item and 48 a record: more than 8 MiB
    one, at = np.ones(n, dtype=np.int32), np.arange(n, dtype=np.int64)
    rpt = torch.tensor([0, 1], dtype=torch.int32, device="cuda").repeat(n)
    cols, vals = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.randn(n, device="cuda")
    hb = K.HostBatch(one, one, one, 2 * at, at, at, at, rpt, cols, vals)
    need = K.bspmm_workspace_bytes(hb, F)
    assert need > 8 << 20
    ws, busy = torch.zeros(need, dtype=torch.uint8, device="cuda"), torch.ones(1 << 28, device="cuda")
    B, C = torch.randn((n, F), device="cuda"), torch.zeros((n, F), device="cuda")
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(60):
            busy.mul_(1.0)                 # the copy waits behind these
    plan = K.bspmm_create(hb, F, None, ws, need, side.cuda_stream)
    K.bspmm_run(plan, B, C, F, F, other.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(C, vals[:, None] * B)
    K.bspmm_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("coo", [False, True])
def test_plan_made_on_another_stream_and_dropped_leaves_no_copy_behind(coo):
    """The workspace goes back to the current stream's allocator: nothing may still be on its way there."""
    import torch
    b = W.random_general(11, 48, [(40, 30, 200), (7, 7, 0), (90, 110, 500)])
    loader = type("Loader", (), dict(vars(b)))()
    if not coo:
        loader.rpt, loader.colids, loader.values = (torch.from_numpy(a).cuda() for a in (b.rpt, b.colids, b.values))
    ids = np.zeros(2 * int(b.nnz.sum()), dtype=np.int32)
    pairs = (torch.from_numpy(ids).cuda(), torch.zeros(int(b.nnz.sum()), device="cuda:0"))
    options = K.make_options(flags=K.COO_DIRECT) if coo else None
    side, busy = torch.cuda.Stream(), torch.randn((4096, 4096), device="cuda:0")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(4):
            busy @ busy
    plan = K.Plan(loader, b.F, options, device="cuda:0", stream=side, coo=pairs if coo else None)
    size, at = plan.workspace.numel(), plan.workspace.data_ptr()
    plan.close()
    del plan
    taken = torch.zeros(size, dtype=torch.uint8, device="cuda:0")
    assert taken.data_ptr() == at
    torch.cuda.synchronize()
    assert not bool(taken.any())


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["converted", "transposed"])
def test_plan_made_on_another_stream_and_dropped_leaves_no_build_behind(kind):
    """As above for what creation enqueues behind the copy: the conversion of index pairs and the
    transposed CSR, both of which write for longer than it takes to clear the memory again."""
    import torch
    b = W.random_general(11, 16, [(400, 300, 6000)] * 600)
    loader = type("Loader", (), dict(vars(b)))()
    loader.rpt, loader.colids, loader.values = (torch.from_numpy(a).cuda() for a in (b.rpt, b.colids, b.values))
    coo = tuple(torch.from_numpy(a).cuda() for a in W.coo_view(b)) if kind == "converted" else None
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    plan = K.Plan(loader, b.F, K.make_options(flags=K.BUILD_TRANSPOSE), device="cuda:0", stream=side, coo=coo)
    size, at = plan.workspace.numel(), plan.workspace.data_ptr()
    plan.close()
    del plan
    taken = torch.zeros(size, dtype=torch.uint8, device="cuda:0")
    assert taken.data_ptr() == at
    torch.cuda.synchronize()
    assert not bool(taken.any())


@pytest.mark.gpu
@pytest.mark.parametrize("coo", [False, True])
def test_plan_made_on_another_stream_waits_for_what_used_its_memory_before(coo):
    """The allocator hands out a block whose last use is still waiting on the current stream."""
    import torch
    from oracle import reference
    b = W.random_general(11, 48, [(40, 30, 200), (7, 7, 0), (90, 110, 500)] * 40)
    C0, S = reference.forward_batch(b)
    loader = type("Loader", (), dict(vars(b)))()
    loader.rpt, loader.colids, loader.values = (torch.from_numpy(a).cuda() for a in (b.rpt, b.colids, b.values))
    pairs = tuple(torch.from_numpy(a).cuda() for a in W.coo_view(b)) if coo else None
    first = K.Plan(loader, b.F, coo=pairs)
    size, at = first.workspace.numel(), first.workspace.data_ptr()
    B, C = torch.from_numpy(b.B).cuda(), torch.zeros((b.n_c_rows, b.F), device="cuda:0")
    side, busy = torch.cuda.Stream(), torch.randn((4096, 4096), device="cuda:0")
    torch.cuda.synchronize()
    first.close()
    del first
    used = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    assert used.data_ptr() == at
    for _ in range(8):
        busy @ busy
    used.fill_(1)                          # waits behind these
    del used
    plan = K.Plan(loader, b.F, device="cuda:0", stream=side, coo=pairs)
    assert plan.workspace.data_ptr() == at
    plan.run(B, C, side)
    torch.cuda.synchronize()
    assert np.all(np.abs(C.cpu().numpy() - C0) <= 1e-5 * S)


@pytest.mark.gpu
def test_native_autograd_is_the_class():
    """batched_spmm on plain tensors gives what BatchedSpMM.apply gives, and leaves to it what it does not take."""
    import torch
    from paper_1903_11409_amd import autograd as A
    b = W.config5_skewed(graphs=40, F=64, asymmetric=True)
    plan = K.Plan(b)
    B = torch.from_numpy(b.B).cuda()
    dY = torch.from_numpy(b.dY).cuda()
    wide = torch.zeros((b.n_b_rows, 80), device="cuda")
    wide[:, :64] = B
    inputs = [B, wide[:, :64], B.t().contiguous().t(), torch.nn.Parameter(B.clone())]
    grads = [dY, torch.ones((1, 1), device="cuda").expand_as(dY), dY.t().contiguous().t()]
    for x in inputs:
        for g in grads:
            out = []
            for f in (A.batched_spmm, A.BatchedSpMM.apply):
                leaf = x.detach().requires_grad_()
                C = f(plan, leaf * 2.0)
                assert C.grad_fn.name() == "BatchedSpMMBackward"
                C.backward(g, retain_graph=True)
                C.backward(g)
                out.append((C.detach(), leaf.grad))
            torch.cuda.synchronize()
            assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    with torch.no_grad():
        assert A.batched_spmm(plan, inputs[3]).grad_fn is None
    assert A.batched_spmm(plan, B, b.n_c_rows + 3).shape == (b.n_c_rows + 3, 64)
    assert not A.batched_spmm(plan, B).requires_grad
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                       # backward on the stream of forward
        leaf = B.clone().requires_grad_()
        A.batched_spmm(plan, leaf).backward(dY)
    side.synchronize()
    assert torch.equal(leaf.grad, plan.run_transposed(dY, torch.empty_like(B)))

    def message(f, *args):
        with pytest.raises(Exception) as e:
            f(plan, *args)
        return str(e.value).splitlines()[0]

    for x in (B.cpu(), B.double(), B[:, :32]):
        assert message(A.batched_spmm, x) == message(A.BatchedSpMM.apply, x)
    under = lambda f: lambda p: torch.func.grad(lambda x: f(p, x).sum())(B)
    assert message(under(A.batched_spmm)) == message(under(A.BatchedSpMM.apply))

    def forward_mode(f):
        def go(p):
            with torch.autograd.forward_ad.dual_level():
                f(p, torch.autograd.forward_ad.make_dual(B, B))
        return go
    assert message(forward_mode(A.batched_spmm)) == message(forward_mode(A.BatchedSpMM.apply))
    C = A.batched_spmm(plan, B.clone().requires_grad_())
    plan.close()
    with pytest.raises(K.BspmmError):
        C.backward(dY)


@pytest.mark.gpu
@pytest.mark.filterwarnings("ignore")
def test_compiled_autograd_traces_the_native_node():
    """A backward pass that compiled autograd traces gives what the class gives there, for plans one after the other."""
    import torch
    import torch._dynamo.compiled_autograd as traced
    from paper_1903_11409_amd import autograd as A
    batches = [W.config5_skewed(seed=s, graphs=20 + s, F=64, asymmetric=True) for s in range(3)]
    results = []
    for f in (A.batched_spmm, A.BatchedSpMM.apply):
        for b in batches + batches[:1]:
            plan = K.Plan(b)
            leaf = torch.from_numpy(b.B).cuda().requires_grad_()
            C = f(plan, leaf * 2.0) + f(plan, leaf)
            with traced._enable(torch.compile(backend="eager")):
                C.backward(torch.from_numpy(b.dY).cuda())
            torch.cuda.synchronize()
            results.append(leaf.grad)
        torch._dynamo.reset()
    for native, of_class in zip(results, results[len(batches) + 1:]):
        assert torch.equal(native, of_class)
    plan = K.Plan(batches[0])
    leaf = torch.from_numpy(batches[0].B).cuda().requires_grad_()
    A.batched_spmm(plan, leaf).backward(torch.from_numpy(batches[0].dY).cuda())
    assert torch.allclose(results[0], 3.0 * leaf.grad, rtol=1e-5, atol=1e-5)
