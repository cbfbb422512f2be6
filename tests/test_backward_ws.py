"""The transposed product through a workspace (es_spmm_backward_ws, which es_spmm_backward of
the Python binding takes for larger sampled products): every element against the oracle at the
sizes where its blocks, walkers and 512-row steps begin and end."""
import numpy as np
import pytest

import paper_2104_10716_amd as es


def test_workspace_is_asked_for_only_where_the_form_applies():
    ask = es.es_spmm_backward_workspace_bytes
    assert ask(170_000, 2_370_240, 128, 16, "bucket") > 16 * 2_370_240          # 16 bytes per kept entry and more
    assert ask(170_000, 2_370_240, 128, 16, "fastrand") == ask(170_000, 2_370_240, 128, 16, "bucket")
    assert ask(170_000, 2_370_240, 128, 0, "full") == 0
    assert ask(170_000, 2_370_240, 17, 16, "bucket") > 0 and ask(170_000, 2_370_240, 16, 16, "bucket") == 0
    assert ask(2 ** 22, 2 ** 24, 64, 16, "bucket") > 0 and ask(2 ** 22 + 1, 2 ** 24, 64, 16, "bucket") == 0
    assert ask(170_000, 2_370_240, 128, 4096, "bucket") > 0 and ask(170_000, 2_370_240, 128, 4097, "bucket") == 0
    assert ask(19_717, 88_000, 32, 16, "bucket") == 0                           # small: the scatter is the faster form
    # 0.7 to 1.1 M requests: the line is on the entries that rows of any length law keep (half of min(nnz, N W) where the
    # two are equal), by requests per entry, and above what two requests per entry repay once there are more rows than threads
    for F, per_entry, need in ((17, 2, 0.52e6), (32, 2, 0.52e6), (33, 3, 0.44e6), (64, 4, 0.44e6), (65, 5, 0.36e6), (256, 16, 0.36e6)):
        for N, W in ((1_500, 200), (10_000, 500), (40_000, 4), (90_000, 4), (262_144, 2)):
            for nnz in [int(x * 1e6 / per_entry) for x in (0.69, 0.71, 0.75, 0.8, 0.9, 1.0, 1.09, 1.11)]:
                most = min(nnz, N * W) * per_entry
                kept = nnz * (N * W) / (nnz + N * W) * per_entry
                taken = most >= 1.1e6 or (most >= 0.7e6 and kept >= need)
                if nnz <= 32 * N or nnz <= N * W:                              # the rule for long rows has no say
                    assert (ask(N, nnz, F, W, "bucket") > 0) == taken, (N, nnz, F, W)
    assert ask(90_000, 360_000, 17, 4, "bucket") == 0 and ask(90_000, 360_000, 65, 4, "bucket") > 0       # 25.9 / 30.6 us at F = 17
    assert ask(262_145, 500_000, 32, 4, "bucket") == 0 and ask(262_145, 500_000, 33, 4, "bucket") > 0
    assert ask(262_145, 550_001, 32, 4, "bucket") > 0
    # few entries kept of long rows: requests per row (W times 2 at F = 32) against the mean row
    assert ask(233_000, 233_000 * 300, 32, 8, "fastrand") == 0 and ask(233_000, 233_000 * 300, 32, 9, "fastrand") > 0
    assert ask(233_000, 233_000 * 300, 32, 4, "bucket") == 0 and ask(233_000, 233_000 * 300, 32, 5, "bucket") > 0
    assert ask(600_000, 600_000 * 33, 32, 3, "fastrand") == 0 and ask(600_000, 600_000 * 32, 32, 3, "fastrand") > 0
    # columns beyond the grid of the gather it ends in (64 at a time on tables of 512 MB and more), or of the scatter
    assert ask(100, 10_000, 65_535 * 64, 100, "bucket") > 0 and ask(100, 10_000, 65_535 * 64 + 1, 100, "bucket") == 0
    assert ask(5, 25, 65_535 * 256, 5, "fastrand") > 0 and ask(5, 25, 65_535 * 256 + 1, 5, "fastrand") == 0
    for bad in ((0, 5, 64, 4), (5, 0, 64, 4), (-1, 5, 64, 4), (1000, 2 ** 31, 64, 10_000), (1000, 10 ** 6, 64, 0)):
        assert ask(*bad, "bucket") == 0


def test_workspace_grows_with_the_entries_kept():
    """16 bytes for each of the min(nnz, N W) entries that can be kept, the counters and the column pointers: no more in
    the one-launch form of the first level, where W may be far above the mean row."""
    ask = es.es_spmm_backward_workspace_bytes
    for N, nnz, F, W in ((16_000, 72_000, 256, 256), (16_000, 240_000, 256, 256), (16_384, 16_384 * 300, 64, 256), (170_000, 2_370_240, 128, 16),
                         (262_144, 262_144 * 5, 32, 16), (1_000, 200_000, 512, 256), (511, 150_000, 256, 200), (65, 4_000, 9_000, 64),
                         (262_145, 262_145 * 5, 32, 16), (40_000, 400_000, 64, 4_096)):
        width = 1
        while width < 1024 and N // (2 * width) >= 1024:
            width *= 2
        blocks, walkers = -(-N // width), min(256, -(-N // 64))
        most = 16 * min(nnz, N * W) + 4 * (walkers * blocks + blocks + 1 + N + 1) + 6 * 255
        assert 16 * min(nnz, N * W) < ask(N, nnz, F, W, "bucket") <= most, (N, nnz, F, W)


def _graph(N, avg, seed, F, ldx=None, hot=None, long_row=0):
    from workloads import random_csr
    rowptr, colidx = random_csr(N, avg, seed, empty_frac=0.05)
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(N), np.diff(rowptr))
    cols = colidx.astype(np.int64)
    if hot is not None:                                # a column that every row holds
        rows, cols = np.concatenate([rows, np.arange(N)]), np.concatenate([cols, np.full(N, hot)])
    if long_row:
        rows = np.concatenate([rows, np.full(long_row, N // 2)])
        cols = np.concatenate([cols, rng.choice(N, long_row, replace=False)])
    key = np.unique(rows * N + cols)
    rowptr = np.zeros(N + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(np.bincount(key // N, minlength=N))
    colidx = (key % N).astype(np.int32)
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    dY = rng.uniform(-1, 1, (N, ldx or F)).astype(np.float32)
    return rowptr, colidx, vals, dY


CASES = [
    # N, avg, F, ldx, mode, W, seed, norm, extras
    (511, 300.0, 256, None, "fastrand", 200, 3, "none", {}),                    # fewer rows than one step, blocks of one column
    (2_047, 90.0, 160, None, "bucket", 64, 0, "mean", {}),
    (2_048, 90.0, 160, 164, "fastrand", 64, 0, "rescale", {}),                    # the first two-column blocks
    (16_385, 14.0, 128, None, "fastrand", 16, 2 ** 63 + 5, "none", {}),         # one row more than all walkers' first
    (40_961, 20.0, 41, 41, "bucket", 33, 0, "inv_degree", {}),                  # rows that are 4-byte aligned only
    (131_073, 9.0, 20, None, "fastrand", 8, 77, "rsqrt", {}),                   # 512 rows and one more per walker
    (30_000, 30.0, 640, 644, "fastrand", 1, 5, "none", dict(hot=29_999)),         # one entry per row; a column of all rows, the last
    (30_000, 25.0, 64, None, "bucket", 16, 0, "none", dict(hot=0)),
    (6_000, 60.0, 64, None, "fastrand", 4_096, 9, "none", dict(long_row=5_900)),  # the widest rows it takes
    (6_000, 60.0, 64, None, "bucket", 4_096, 0, "none", dict(long_row=4_097)),
    # rows far longer than W: every transposed row that is not empty is longer than four times their mean
    (9_001, 390.0, 128, None, "bucket", 22, 0, "mean", {}),
    (30_000, 230.0, 20, None, "bucket", 24, 0, "none", dict(hot=0)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("N,avg,F,ldx,mode,W,seed,norm,extra", CASES)
def test_backward_through_a_workspace(N, avg, F, ldx, mode, W, seed, norm, extra):
    import torch
    from gpu_util import DeviceCSR, check_Y, check_backward_against_oracle
    import oracle
    rowptr, colidx, vals, dY = _graph(N, avg, N + F, F, ldx, **extra)
    nbytes = es.es_spmm_backward_workspace_bytes(N, colidx.size, F, W, mode)
    assert nbytes > 0
    for v in (vals, None):
        d = DeviceCSR(rowptr, colidx, v, dY, F=F)
        what = f"N={N} F={F} {mode} W={W} {norm}"
        check_backward_against_oracle(d, W, mode, seed, norm, what=what)        # torch's allocator lends the workspace
        ref, den = oracle.spmm_backward(rowptr, colidx, v, dY, F, W, mode, seed, norm=norm)
        for size in (nbytes, nbytes - 256):                                     # its own, and one that is too small: the scatter
            ws = torch.full((size // 4,), -1, dtype=torch.int32, device="cuda:0")
            dX = torch.full((N, F + 3), float("nan"), dtype=torch.float32, device="cuda:0")
            es.es_spmm_backward_ws(d.rowptr, d.colidx, d.vals, d.X, dX, W, mode, seed, norm, ws, F=F)
            torch.cuda.synchronize()
            assert torch.isnan(dX[:, F:]).all()
            check_Y(dX[:, :F].cpu().numpy(), ref, den, f"{what} workspace {size}")


@pytest.mark.gpu
@pytest.mark.parametrize("N,avg,F,ldx,mode,W,seed,norm,extra", [
    # walkers whose entries fit their registers, at most 1024 rows and 16 entries per thread, and just no longer
    (16_384, 20.0, 64, None, "fastrand", 256, 3, "mean", dict(long_row=9_000)), (16_384, 20.0, 64, None, "fastrand", 257, 3, "mean", {}),
    (16_384, 260.0, 20, None, "bucket", 256, 0, "none", {}),                     # every place of a walker taken
    (262_144, 4.0, 20, None, "bucket", 16, 0, "none", dict(hot=262_143)), (262_145, 4.0, 20, None, "fastrand", 16, 9, "none", {}),
    (1_000, 200.0, 512, None, "fastrand", 256, 2 ** 63 + 5, "rescale", {}), (65, 60.0, 9_000, None, "bucket", 64, 0, "none", {}),
    (2_048, 300.0, 160, 164, "fastrand", 257, 7, "none", {}), (40_961, 130.0, 41, 41, "bucket", 120, 0, "inv_degree", {}),
    (131_073, 40.0, 20, None, "fastrand", 33, 77, "rsqrt", {})])
def test_backward_through_a_workspace_around_what_a_walker_holds(N, avg, F, ldx, mode, W, seed, norm, extra):
    test_backward_through_a_workspace(N, avg, F, ldx, mode, W, seed, norm, extra)


@pytest.mark.gpu
@pytest.mark.parametrize("N,avg,F,mode,W,more", [
    (16_384, 4.5, 256, "fastrand", 256, 0), (16_384, 4.5, 256, "fastrand", 256, 977_777),      # rows far shorter than W
    (30_000, 60.0, 41, "bucket", 16, 0), (30_000, 60.0, 41, "bucket", 16, 5), (262_144, 3.0, 20, "bucket", 5, 0),
    (16_385, 4.5, 256, "fastrand", 256, 0)])                                                   # more than a walker holds
def test_backward_workspace_is_not_written_beyond_its_size(N, avg, F, mode, W, more):
    """A walker's records lie where its rows' entries can at most begin; nnz (the length of colidx) may be more
    than rowptr[N]."""
    import torch
    from gpu_util import DeviceCSR, check_Y
    import oracle
    rowptr, colidx, vals, dY = _graph(N, avg, N + F, F, long_row=3_000)
    nnz = colidx.size + more
    nbytes = es.es_spmm_backward_workspace_bytes(N, nnz, F, W, mode)
    assert nbytes > 0
    d = DeviceCSR(rowptr, colidx, vals, dY)
    longer, values = (torch.cat([t, t.new_zeros(more)]) for t in (d.colidx, d.vals))
    whole = torch.full((nbytes // 4 + 4_096,), -7, dtype=torch.int32, device="cuda:0")
    dX = torch.full((N, F), float("nan"), dtype=torch.float32, device="cuda:0")
    es.es_spmm_backward_ws(d.rowptr, longer, values, d.X, dX, W, mode, 5, "none", whole[:nbytes // 4])
    torch.cuda.synchronize()
    assert bool((whole[nbytes // 4:] == -7).all()) and not bool((whole[:nbytes // 4] == -7).all())
    check_Y(dX.cpu().numpy(), *oracle.spmm_backward(rowptr, colidx, vals, dY, F, W, mode, 5), f"N={N} W={W} nnz + {more}")


@pytest.mark.gpu
def test_backward_workspace_on_streams_in_graphs_and_with_infinities():
    import torch
    from gpu_util import DeviceCSR, check_Y
    import oracle
    N, F, W = 20_000, 64, 16
    rowptr, colidx, vals, dY = _graph(N, 20.0, 5, F)
    d = DeviceCSR(rowptr, colidx, vals, dY)
    ref, den = oracle.spmm_backward(rowptr, colidx, vals, dY, F, W, "fastrand", 3)
    assert es.es_spmm_backward_workspace_bytes(N, colidx.size, F, W, "fastrand") > 0
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    outs = [torch.full((N, F), float("nan"), device="cuda:0") for _ in range(4)]
    side.wait_stream(torch.cuda.current_stream())
    for out, s in zip(outs, (None, side, side.cuda_stream, None)):              # calls on two streams, each with scratch of its own
        es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, out, W, "fastrand", 3, stream=s, nnz=7)   # nnz: only a hint here
    torch.cuda.synchronize()
    for out in outs:
        check_Y(out.cpu().numpy(), ref, den, "streams")
    with pytest.raises(es.EsSpmmError):                # a hint that the scatter refuses is refused here too
        es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, outs[0], W, "fastrand", 3, nnz=-1)
    # inside a graph the form without a workspace runs; every replay is whole
    with torch.cuda.stream(side):
        es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, outs[0], W, "fastrand", 3)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, outs[1], W, "fastrand", 3)
    for _ in range(3):
        outs[1].fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        check_Y(outs[1].cpu().numpy(), ref, den, "replay")
    # an infinite or missing gradient reaches the same places as by the scatter, and no others
    d.X[11, 5], d.X[4_000, 6] = float("inf"), float("nan")
    es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, outs[2], W, "fastrand", 3)
    es.es_spmm_backward_ex(d.rowptr, d.colidx, d.vals, d.X, outs[3], W, "fastrand", 3)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(outs[2]), torch.isnan(outs[3]))
    assert torch.equal(torch.isposinf(outs[2]), torch.isposinf(outs[3]))
    assert torch.equal(torch.isneginf(outs[2]), torch.isneginf(outs[3]))
    assert int(torch.isinf(outs[2]).sum()) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("N", [2 ** 22 - 1_024, 2 ** 22 - 1_023, 2 ** 22])
def test_backward_workspace_with_the_most_column_blocks(N):
    """4095 and 4096 blocks of 1024 columns, the last of them whole or of one column: one entry per row, any
    column, against the same sum in 64 bits."""
    import torch
    F = 17
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(N)
    rowptr = torch.arange(N + 1, dtype=torch.int32, device=dev)
    colidx = torch.randint(N, (N,), device=dev, generator=gen)
    colidx[-1] = N - 1
    vals = torch.randn(N, device=dev, generator=gen)
    dY = torch.randn(N, F, device=dev, generator=gen)
    assert es.es_spmm_backward_workspace_bytes(N, N, F, 1, "fastrand") > 0
    dX = es.es_spmm_backward(rowptr, colidx.int(), vals, dY, torch.full_like(dY, float("nan")), 1, "fastrand", 3)
    terms = vals.double()[:, None] * dY.double()
    ref, den = (torch.zeros(N, F, dtype=torch.float64, device=dev).index_add_(0, colidx, t) for t in (terms, terms.abs()))
    assert bool(((dX.double() - ref).abs() <= 1e-5 * den).all())


@pytest.mark.gpu
def test_backward_workspace_beside_another_threads_capture():
    """The first call in a thread takes its workspace while another thread captures a graph: the
    capture and the call both come out whole."""
    import threading
    import torch
    from gpu_util import DeviceCSR, check_Y
    import oracle
    N, F, W = 20_000, 64, 16
    rowptr, colidx, vals, dY = _graph(N, 20.0, 5, F)
    d = DeviceCSR(rowptr, colidx, vals, dY)
    ref, den = oracle.spmm_backward(rowptr, colidx, vals, dY, F, W, "bucket")
    assert es.es_spmm_backward_workspace_bytes(N, colidx.size, F, W, "bucket") > 0
    side = torch.cuda.Stream()
    out, captured = (torch.full((N, F), float("nan"), device="cuda:0") for _ in range(2))
    es.es_spmm(d.rowptr, d.colidx, d.vals, d.X, captured, W, "bucket")
    torch.cuda.synchronize()
    expected = captured.clone()
    failed = []

    def call():
        try:
            es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, out, W, "bucket", stream=side)
        except Exception as e:                         # noqa: BLE001 (reported below)
            failed.append(e)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):                      # empties torch's cache of memory, then captures in global mode
        es.es_spmm(d.rowptr, d.colidx, d.vals, d.X, captured, W, "bucket")
        t = threading.Thread(target=call)
        t.start()
        t.join()
    assert not failed, failed
    torch.cuda.synchronize()
    check_Y(out.cpu().numpy(), ref, den, "beside a capture")
    for _ in range(3):
        captured.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured, expected)


@pytest.mark.gpu
def test_backward_workspace_with_as_many_entries_as_int32_counts():
    """2^31 - 128 kept entries: the last column block ends within one step of the largest index.
    Row r holds columns r .. r + 4094 (mod N), so a row of dX is a window of dY, summed here in 64 bits."""
    import torch
    N, K, F = 524_416, 4_095, 17
    assert 2 ** 31 - 8 * 256 < N * K < 2 ** 31
    dev = torch.device("cuda:0")
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    rowptr = torch.arange(N + 1, dtype=torch.int32, device=dev) * K
    colidx = torch.empty(N * K, dtype=torch.int32, device=dev)
    window = torch.arange(K, dtype=torch.int32, device=dev)
    for r in range(0, N, 65_536):
        rows = torch.arange(r, min(N, r + 65_536), dtype=torch.int32, device=dev)
        part = (rows[:, None] + window).remainder_(N)
        colidx[r * K:r * K + part.numel()] = part.view(-1)
    del part
    gen = torch.Generator(device=dev).manual_seed(3)
    dY = torch.randn(N, F, device=dev, generator=gen)
    nbytes = es.es_spmm_backward_workspace_bytes(N, N * K, F, 4_096, "bucket")
    assert nbytes > 16 * N * K
    ws = torch.empty(nbytes // 4, dtype=torch.int32, device=dev)
    dX = torch.full((N, F), float("nan"), device=dev)
    print("  2^31 - 128 entries: launching", flush=True)
    es.es_spmm_backward_ws(rowptr, colidx, None, dY, dX, 4_096, "bucket", workspace=ws)
    torch.cuda.synchronize()

    def window_sums(t):                                # row c: the sum of rows c - 4094 .. c (mod N)
        run = torch.cat([t[N - K + 1:], t]).double().cumsum(0)
        return run[K - 1:] - torch.cat([run.new_zeros(1, F), run[:N - 1]])
    err = (dX.double() - window_sums(dY)).abs()
    assert bool((err <= 1e-5 * window_sums(dY.abs())).all())
