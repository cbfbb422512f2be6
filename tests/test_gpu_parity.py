"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the
same seeded inputs -- sampled edge lists bit-exact, Y within the normalised
1e-5 bound.  Needs an MI355X; run with -m gpu."""
import ctypes
import functools
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def es():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2104_10716_amd as es
    es.load_library()          # raises if the HIP library is missing: no fallback
    return es


@functools.lru_cache(maxsize=2)
def _workload(cfg):
    from workloads import make_workload
    return make_workload(cfg)


def _random_graph(n, avg, seed, F, ldx=None, empty_frac=0.1, unit_vals=False):
    from workloads import random_csr
    rowptr, colidx = random_csr(n, avg, seed, empty_frac=empty_frac)
    rng = np.random.default_rng(seed + 1)
    vals = None if unit_vals else rng.standard_normal(colidx.size).astype(np.float32)
    ldx = F if ldx is None else ldx
    X = rng.uniform(-1, 1, (n, ldx)).astype(np.float32)
    return rowptr, colidx, vals, X


# --------------------------------------------------------------------------
# small graphs: every mode, ragged shapes, every launch shape
# --------------------------------------------------------------------------
@pytest.mark.parametrize("F,ldx", [(1, 1), (3, 5), (4, 4), (16, 16), (17, 20), (41, 41), (64, 64),
                                   (100, 128), (128, 128), (130, 130), (256, 256), (260, 260),
                                   (602, 602), (1028, 1028)])
def test_small_graph_all_modes(es, F, ldx):
    from gpu_util import DeviceCSR, check_against_oracle, check_edges
    n = 777                                    # ragged: not a multiple of any tile
    rowptr, colidx, vals, X = _random_graph(n, 9.0, seed=F, F=F, ldx=ldx)
    d = DeviceCSR(rowptr, colidx, vals, X, F=F)
    maxdeg = int(np.diff(rowptr).max())
    _say(f"small graph F={F} ldx={ldx} maxdeg={maxdeg}")
    for rpw in (0, 1, 4, 64):
        opts = dict(rows_per_wave=rpw) if rpw else None      # None: the plain es_spmm entry point
        check_against_oracle(d, 0, "full", what=f"full F={F} rpw={rpw}", opts=opts)
        for mode in ("bucket", "fastrand"):
            for W in (1, 3, 8, maxdeg, maxdeg + 5):
                for seed in (0, 12345):
                    check_against_oracle(d, W, mode, seed, ldy=ldx + 4 if F % 4 == 0 else None,
                                         what=f"{mode} F={F} W={W} seed={seed} rpw={rpw}", opts=opts)
    # the flattened kernel (needs 128-bit accesses: F >= 4), whole and sliced, with and without long rows
    if F >= 4:
        for opts in (dict(kernel=2), dict(kernel=2, lanes_per_row=4), dict(kernel=2, lanes_per_row=8),
                     dict(kernel=2, long_row_threshold=5)):
            info = es.es_spmm_launch_info(n, colidx.size, F, 3, "fastrand", ldx=ldx, ldy=ldx, opts=opts,
                                          aligned16=(F % 4 == 0 and ldx % 4 == 0))
            assert info["flattened"] == 1
            check_against_oracle(d, 0, "full", what=f"flattened full F={F} {opts}", opts=opts)
            for mode in ("bucket", "fastrand"):
                for W in (1, 3, 8, maxdeg, maxdeg + 5):
                    for seed in (0, 12345):
                        check_against_oracle(d, W, mode, seed, ldy=ldx + 4 if F % 4 == 0 else None, norm="rescale",
                                             what=f"flattened {mode} F={F} W={W} seed={seed} {opts}", opts=opts)
    # force the long-row path (segments + atomic adds) onto ordinary rows
    for thr in (1, 7):
        opts = dict(long_row_threshold=thr)
        check_against_oracle(d, 0, "full", what=f"full F={F} long-row threshold {thr}", opts=opts)
        for mode in ("bucket", "fastrand"):
            check_against_oracle(d, maxdeg - 1, mode, 12345, what=f"{mode} F={F} long-row threshold {thr}",
                                 opts=opts)
    for mode in ("bucket", "fastrand"):
        for W in (1, 3, 8, maxdeg):
            for rpw in (0, 1, 2, 8, 64, -1):
                check_edges(d, W, mode, 12345, rpw)


@pytest.mark.parametrize("F", [64, 100, 256, 520])
def test_column_slicing_override(es, F):
    """lanes_per_row option: narrower column blocks (several per row, the
    sampler evaluated once per block) must give the same product."""
    from gpu_util import DeviceCSR, check_against_oracle
    rowptr, colidx, vals, X = _random_graph(900, 14.0, seed=F + 7, F=F, ldx=F + (4 - F % 4) % 4)
    d = DeviceCSR(rowptr, colidx, vals, X, F=F)
    for lanes in (4, 8, 16, 32, 64, 0, -1):
        for thr in (0, 6):
            opts = dict(lanes_per_row=lanes, long_row_threshold=thr)
            for mode, W in (("full", 0), ("bucket", 5), ("fastrand", 5), ("fastrand", 25)):
                check_against_oracle(d, W, mode, 3, norm="mean", opts=opts,
                                     what=f"lanes={lanes} thr={thr} F={F} {mode} W={W}")


@pytest.mark.parametrize("F,ldx", [(1, 1), (4, 4), (17, 20), (41, 41), (64, 64), (100, 128), (128, 128),
                                   (260, 260), (602, 602)])
def test_column_partitioned_product(es, F, ldx):
    """es_spmm_ws with the column-partitioned product forced on: eight launches
    that each add one column range's share of every row must give the oracle's
    product, for every launch shape, row factor and output stride."""
    from gpu_util import DeviceCSR, check_against_oracle
    n = 1531                                   # not a multiple of 8, of the row blocks or of any tile
    rowptr, colidx, vals, X = _random_graph(n, 40.0, seed=300 + F, F=F, ldx=ldx)
    d = DeviceCSR(rowptr, colidx, vals, X, F=F)
    maxdeg = int(np.diff(rowptr).max())
    _say(f"column-partitioned F={F} ldx={ldx} maxdeg={maxdeg}")
    for rpw in (0, 1, 4, 64):
        for lanes, thr, kern in ((0, 0, 1), (8, 0, 1), (0, 2, 1), (0, 10 ** 6, 1), (0, 0, 2), (8, 0, 2), (4, 0, 2)):
            if kern == 2 and (F < 4 or rpw):                          # thr: pieces above it go to the first sweep
                continue
            opts = dict(workspace=True, column_partition=1, rows_per_wave=rpw, lanes_per_row=lanes,
                        long_row_threshold=thr, kernel=kern)
            info = es.es_spmm_launch_info(n, colidx.size, F, 8, "fastrand", ldx=ldx, ldy=ldx + 4,
                                          opts={k: v for k, v in opts.items() if k != "workspace"})
            assert info["column_ranges"] == 8
            assert info["long_row_workgroups"] * 2 == info["grid_x"] or info["flattened"]
            check_against_oracle(d, 0, "full", what=f"partitioned full F={F} rpw={rpw} lanes={lanes}", opts=opts)
            for W in (1, 7, 30, maxdeg - 1, maxdeg + 5):
                for seed in (0, 12345):
                    check_against_oracle(d, W, "fastrand", seed, ldy=ldx + 4 if F % 4 == 0 else None,
                                         norm="mean" if seed else None, opts=opts,
                                         what=f"partitioned fastrand F={F} W={W} seed={seed} rpw={rpw} lanes={lanes}")
            # Bucket never takes the partitioned path: same call, plain product
            check_against_oracle(d, 7, "bucket", 0, what=f"bucket with a workspace F={F}", opts=opts)
    # a workspace that is too small, or none: the plain product
    import torch
    small = torch.empty(8, dtype=torch.int32, device="cuda:0")
    check_against_oracle(d, 0, "full", what="workspace too small", opts=dict(workspace=small, column_partition=1))
    check_against_oracle(d, 0, "full", what="no workspace", opts=dict(workspace=None, column_partition=1))
    assert es.es_spmm_workspace_bytes(n) == 4 * 8 * n


def test_column_partitioned_product_edge_cases(es):
    """Rows out of column order (the pieces found by binary search must still
    tile every row), duplicate columns, empty rows, all entries in one column
    range, long rows spanning several tiles."""
    import torch
    from gpu_util import DeviceCSR, check_against_oracle
    rng = np.random.default_rng(8)
    n = 2000
    rowptr, colidx, vals, X = _random_graph(n, 60.0, seed=77, F=32, empty_frac=0.2)
    force = dict(workspace=True, column_partition=1)
    # (a) one single row out of order
    ci = colidx.copy()
    r = int(np.argmax(np.diff(rowptr) > 5))
    ci[[rowptr[r], rowptr[r] + 3]] = ci[[rowptr[r] + 3, rowptr[r]]]
    d = DeviceCSR(rowptr, ci, vals, X)
    for mode, W in (("full", 0), ("fastrand", 9), ("fastrand", 200)):
        check_against_oracle(d, W, mode, 3, what=f"one row out of order {mode} W={W}", opts=force)
    # (b) every row shuffled
    ci = colidx.copy()
    for r in range(n):
        rng.shuffle(ci[rowptr[r]:rowptr[r + 1]])
    d = DeviceCSR(rowptr, ci, vals, X)
    for mode, W in (("full", 0), ("fastrand", 9)):
        check_against_oracle(d, W, mode, 3, what=f"shuffled rows {mode} W={W}", opts=force)
    # (c) duplicate columns inside rows (non-decreasing, not strictly increasing)
    ci = colidx.copy()
    dup = rng.random(colidx.size) < 0.3
    dup[rowptr[:-1][np.diff(rowptr) > 0]] = False         # never a row's first entry
    for p in np.nonzero(dup)[0]:
        ci[p] = ci[p - 1]                                  # in order: runs of equal columns
    d = DeviceCSR(rowptr, ci, vals, X)
    for mode, W in (("full", 0), ("fastrand", 9)):
        check_against_oracle(d, W, mode, 3, what=f"duplicate columns {mode} W={W}", opts=force)
    # (d) all columns inside one range (range 5 of 8), and rows of 0 .. 3000 entries
    lengths = [0, 1, 63, 64, 65, 511, 512, 513, 577, 1154, 3000, 2999] * 60
    N = len(lengths)
    lo, hi = 5 * ((N + 7) // 8), min(N, 6 * ((N + 7) // 8))
    cols = [np.sort(rng.integers(lo, hi, size=L)) for L in lengths]
    rp = np.zeros(N + 1, dtype=np.int32)
    rp[1:] = np.cumsum(lengths)
    cc = np.concatenate(cols).astype(np.int32)
    vv = rng.standard_normal(cc.size).astype(np.float32)
    XX = rng.uniform(-1, 1, (N, 16)).astype(np.float32)
    d = DeviceCSR(rp, cc, vv, XX)
    for rpw in (0, 1, 8):
        opts = dict(force, rows_per_wave=rpw)
        check_against_oracle(d, 0, "full", what=f"one column range, full, rpw={rpw}", opts=opts)
        for W in (16, 512, 600, 1153, 2999):
            check_against_oracle(d, W, "fastrand", 5, what=f"one column range, fastrand W={W} rpw={rpw}", opts=opts)
    # (e) the workspace is reused across calls without being cleared in between
    ws = torch.full((es.es_spmm_workspace_bytes(n) // 4,), 0x7FFFFFFF, dtype=torch.int32, device="cuda:0")
    d = DeviceCSR(rowptr, colidx, vals, X)
    for rep in range(2):
        check_against_oracle(d, 0, "full", what="shared workspace, sorted graph", opts=dict(force, workspace=ws))
        ci2 = colidx.copy()
        for r in range(n):
            rng.shuffle(ci2[rowptr[r]:rowptr[r + 1]])
        check_against_oracle(DeviceCSR(rowptr, ci2, vals, X), 0, "full", what="shared workspace, shuffled graph",
                             opts=dict(force, workspace=ws))


def test_randomised_shapes(es):
    """Seeded sweep over random combinations of graph size, degree, F, row
    strides, W, mode, seed, row factor and the per-call launch options, forward
    and transposed, each against the oracle."""
    import torch
    from gpu_util import DeviceCSR, check_against_oracle, check_backward_against_oracle, check_edges
    rng = np.random.default_rng(20260101)
    for case in range(400):
        n = int(rng.choice([1, 2, 63, 64, 65, 257, 1000, 3001]))
        avg = float(rng.choice([0.5, 3.0, 20.0, 90.0]))
        F = int(rng.choice([1, 2, 4, 5, 8, 12, 16, 31, 32, 41, 64, 96, 100, 128, 192, 256, 300, 512, 700]))
        pad = int(rng.choice([0, 0, 1, 3, 4]))
        rowptr, colidx, vals, X = _random_graph(n, avg, seed=1000 + case, F=F, ldx=F + pad,
                                                empty_frac=float(rng.choice([0.0, 0.3])),
                                                unit_vals=bool(rng.integers(0, 4) == 0))
        d = DeviceCSR(rowptr, colidx, vals, X, F=F)
        maxdeg = max(1, int(np.diff(rowptr).max()))
        mode = str(rng.choice(["full", "bucket", "fastrand", "fastrand"]))
        W = int(rng.choice([1, 2, 7, 16, 33, max(1, maxdeg - 1), maxdeg, maxdeg + 9]))
        seed = int(rng.choice([0, 1, 2 ** 63 + 12345]))
        norm = str(rng.choice(["none", "none", "mean", "rsqrt", "rescale", "inv_degree"]))
        rpw = int(rng.choice([0, 0, 1, 2, 16, 64]))
        thr = int(rng.choice([0, 0, 1, 3, 40]))
        lanes = int(rng.choice([0, 0, 0, 4, 16]))
        opts = dict(rows_per_wave=rpw, long_row_threshold=thr, lanes_per_row=lanes, kernel=int(rng.choice([0, 1, 2])))
        part = int(rng.choice([0, 0, 1, -1]))
        if part:
            opts.update(workspace=True, column_partition=part)
        what = (f"case {case}: part={part} kernel={opts['kernel']} n={n} avg={avg} F={F} ld={F + pad} {mode} W={W} seed={seed} norm={norm} "
                f"rpw={rpw} thr={thr} lanes={lanes}")
        _say(what)
        ldy = F + int(rng.choice([0, 0, 2, 4]))
        check_against_oracle(d, W, mode, seed, ldy=ldy, norm=norm, what=what, opts=opts)
        opts.pop("workspace", None)
        check_backward_against_oracle(d, W, mode, seed, norm, what="backward " + what, opts=opts)
        if mode != "full":
            check_edges(d, W, mode, seed, int(rng.choice([0, 1, 4, -1])), what="edges " + what)


@pytest.mark.parametrize("ld", [1 << 20, (1 << 20) + 1])
def test_row_offsets_beyond_32_bits(es, ld):
    """A dense matrix whose largest row offset does not fit 32 bits (5 000 rows at
    a row stride of 2^20 floats: 21 GB, touched sparsely) takes the kernels that
    multiply column ids by the stride in 64 bits; same products, forward, column-
    partitioned and transposed."""
    import torch
    import oracle
    from gpu_util import check_Y
    n, F = 5000, 8
    rowptr, colidx, vals, Xh = _random_graph(n, 12.0, seed=ld % 97, F=F)
    dev = "cuda:0"
    big = torch.empty(n * ld, dtype=torch.float32, device=dev)
    X = big.as_strided((n, F), (ld, 1))
    X.copy_(torch.from_numpy(Xh))
    rp, ci, va = (torch.from_numpy(a).to(dev) for a in (rowptr, colidx, vals))
    Y = torch.empty((n, F), dtype=torch.float32, device=dev)
    ws = torch.empty(es.es_spmm_workspace_bytes(n) // 4, dtype=torch.int32, device=dev)
    for mode, W, opts in (("full", 0, None), ("fastrand", 5, None), ("bucket", 5, dict(long_row_threshold=3)),
                          ("full", 0, dict(column_partition=1)), ("fastrand", 5, dict(column_partition=1)),
                          ("full", 0, dict(kernel=2)), ("fastrand", 5, dict(kernel=2)), ("bucket", 5, dict(kernel=2)),
                          ("full", 0, dict(kernel=2, column_partition=1))):        # flattened kernel, wide keys
        Y.fill_(float("nan"))
        es.es_spmm_ws(rp, ci, va, X, Y, W, mode, 3, "none", opts, ws)
        torch.cuda.synchronize()
        Yref, den = oracle.spmm(rowptr, colidx, vals, Xh, F, W, mode, 3)
        check_Y(Y.cpu().numpy(), Yref, den, f"wide row offsets ld={ld} {mode} W={W} opts={opts}")
    # transposed product: the OUTPUT has the wide stride
    dY = torch.from_numpy(Xh).to(dev)
    big.zero_()
    es.es_spmm_backward(rp, ci, va, dY, X, 5, "fastrand", 3)
    torch.cuda.synchronize()
    ref, den = oracle.spmm_backward(rowptr, colidx, vals, Xh, F, 5, "fastrand", 3)
    check_Y(X.cpu().numpy(), ref, den, f"wide row offsets ld={ld} backward")
    del big, X
    torch.cuda.empty_cache()


@pytest.mark.parametrize("ld", [1 << 30, (1 << 30) + 1, (1 << 30) + 1024])
def test_row_strides_whose_bytes_exceed_32_bits(es, ld):
    """Row strides of 4 GiB and a little more (the C ABI takes any 31-bit ldx):
    the bytes from one row of X to the next do not fit 32 bits either.  Three
    rows, 8.6 GB touched sparsely, every forward kernel."""
    import torch
    import oracle
    from gpu_util import check_Y
    n, F = 3, 16
    rowptr = np.array([0, 3, 4, 6], dtype=np.int32)
    colidx = np.array([0, 1, 2, 1, 0, 2], dtype=np.int32)
    rng = np.random.default_rng(ld % 97)
    vals = rng.standard_normal(6).astype(np.float32)
    Xh = rng.uniform(-1, 1, (n, F)).astype(np.float32)
    dev = "cuda:0"
    X = torch.empty((n - 1) * ld + F, dtype=torch.float32, device=dev).as_strided((n, F), (ld, 1))
    X.copy_(torch.from_numpy(Xh))
    rp, ci, va = (torch.from_numpy(a).to(dev) for a in (rowptr, colidx, vals))
    for kernel in (0, 1, 2):
        for mode, W, thr in (("full", 0, 0), ("full", 0, 2), ("bucket", 2, 0), ("fastrand", 2, 0), ("fastrand", 2, 1)):
            what = f"ld={ld} kernel={kernel} {mode} W={W} long rows above {thr}"
            _say(what)
            Y = torch.full((n, F), float("nan"), device=dev)
            es.es_spmm_ex(rp, ci, va, X, Y, W, mode, 3, "none", dict(kernel=kernel, long_row_threshold=thr))
            torch.cuda.synchronize()
            Yref, den = oracle.spmm(rowptr, colidx, vals, Xh, F, W, mode, 3)
            check_Y(Y.cpu().numpy(), Yref, den, what)
    del X
    torch.cuda.empty_cache()


def test_long_rows_span_several_tiles(es):
    """Rows far longer than one LDS tile (full mode and W above the tile),
    including lengths that are multiples of 577 where the multiplier changes."""
    from gpu_util import DeviceCSR, check_against_oracle, check_edges
    n = 6000
    lengths = [0, 1, 5, 511, 512, 513, 577, 1154, 2 * 577 * 2, 1500, 4097, 5999, 64, 63, 65, 1023]
    rng = np.random.default_rng(5)
    cols = [np.sort(rng.choice(n, size=L, replace=False)) for L in lengths]
    reps = 6
    rowptr = np.zeros(len(lengths) * reps + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum([len(c) for c in cols] * reps)
    colidx = np.concatenate(cols * reps).astype(np.int32)
    N = len(lengths) * reps
    # square matrix: pad with empty rows up to n
    rowptr = np.concatenate([rowptr, np.full(n - N, rowptr[-1], dtype=np.int32)])
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    for F in (16, 64, 41):
        X = rng.uniform(-1, 1, (n, F)).astype(np.float32)
        d = DeviceCSR(rowptr, colidx, vals, X)
        for rpw in (0, 1, 4, 16):
            opts = dict(rows_per_wave=rpw)
            _say(f"long rows F={F} rpw={rpw}")
            check_against_oracle(d, 0, "full", what=f"long full F={F} rpw={rpw}", opts=opts)
            for W in (16, 512, 576, 600, 1153, 3000):
                for mode in ("bucket", "fastrand"):
                    check_against_oracle(d, W, mode, 77, what=f"long {mode} F={F} W={W} rpw={rpw}", opts=opts)
        for opts in (dict(kernel=2), dict(kernel=2, long_row_threshold=600), dict(kernel=2, lanes_per_row=4)):
            check_against_oracle(d, 0, "full", what=f"long full F={F} {opts}", opts=opts)
            for W in (16, 512, 576, 600, 1153, 3000):
                for mode in ("bucket", "fastrand"):
                    check_against_oracle(d, W, mode, 77, what=f"long {mode} F={F} W={W} {opts}", opts=opts)
        for thr in (100, 512, 1000, 5000):  # move the long-row threshold around
            opts = dict(long_row_threshold=thr)
            check_against_oracle(d, 0, "full", what=f"long full F={F} threshold {thr}", opts=opts)
            for W in (600, 1153, 3000):
                check_against_oracle(d, W, "fastrand", 77, what=f"long fastrand F={F} W={W} threshold {thr}",
                                     opts=opts)
    for W in (16, 512, 576, 600, 1153, 3000):
        for rpw in (0, 1, 8, -1):
            for seed in (0, 77):
                check_edges(d, W, "fastrand", seed, rpw)
                check_edges(d, W, "bucket", seed, rpw)


@pytest.mark.parametrize("F,lanes", [(16, 0), (32, 0), (64, 0), (64, 8), (128, 0), (128, 8), (256, 0), (41, 0)])
def test_flattened_kernel_rows_at_tile_boundaries(es, F, lanes):
    """The flattened kernel on row lengths around everything it counts in: the
    edge slots of a step (1..16), a batch (64), a tile (256) and several tiles,
    empty rows in runs, in an order that puts row starts and ends on and next to
    tile boundaries; every mode, whole rows and column-range pieces."""
    from gpu_util import DeviceCSR, check_against_oracle
    n = 1200
    rng = np.random.default_rng(900 + F + lanes)
    menu = [0, 0, 0, 1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193,
            255, 256, 257, 300, 511, 512, 513, 767, 768, 769, 1000, 1100]
    for variant in range(3):
        lengths = list(rng.permutation(menu * 2))
        if variant == 1:                      # exact fills: runs that end on a tile boundary
            lengths = [256, 0, 0, 128, 128, 64, 64, 64, 64, 0, 512, 8, 248, 16, 240, 1, 255] * 3
        if variant == 2:                      # nothing but empty rows, then one entry at the very end
            lengths = [0] * 150 + [1]
        cols = [np.sort(rng.choice(n, size=int(L), replace=False)) for L in lengths]
        rowptr = np.zeros(n + 1, dtype=np.int32)
        rowptr[1:len(lengths) + 1] = np.cumsum([len(c) for c in cols])
        rowptr[len(lengths) + 1:] = rowptr[len(lengths)]
        colidx = np.concatenate(cols).astype(np.int32)
        vals = rng.standard_normal(colidx.size).astype(np.float32)
        X = rng.uniform(-1, 1, (n, F)).astype(np.float32)
        d = DeviceCSR(rowptr, colidx, vals, X).with_workspace()
        base = dict(kernel=2, workspace=d.default_ws)
        if lanes:
            base["lanes_per_row"] = lanes
        _say(f"tile boundaries F={F} lanes={lanes} variant {variant}")
        for extra in (dict(), dict(long_row_threshold=700), dict(column_partition=1)):
            opts = dict(base, **extra)
            info = es.es_spmm_launch_info(n, colidx.size, F, 0, "full", aligned16=(F % 4 == 0),
                                          opts={k: v for k, v in opts.items() if k != "workspace"})
            assert info["flattened"] == 1, info
            check_against_oracle(d, 0, "full", what=f"full F={F} {extra} variant {variant}", opts=opts)
            for mode in ("bucket", "fastrand"):
                for W in (1, 7, 8, 64, 255, 256, 257, 1024):
                    for seed in (0, 99):
                        check_against_oracle(d, W, mode, seed, norm="mean",
                                             what=f"{mode} W={W} seed={seed} F={F} {extra} variant {variant}",
                                             opts=opts)


@pytest.mark.parametrize("F,lanes", [(16, 0), (64, 8), (64, 0), (128, 0), (256, 0), (41, 0)])
@pytest.mark.parametrize("ld", [0, 1 << 22])
def test_flattened_kernel_absent_entries_multiply_nothing(es, F, lanes, ld):
    """Infinities in X: a row of Y holds one exactly where the sum of its own kept entries
    does, whatever the flattened kernel pads the row with (64-bit offsets too: ld = 2^22)."""
    import torch
    from gpu_util import DeviceCSR
    n = 60
    rng = np.random.default_rng(F + lanes)
    lengths = rng.permutation(np.concatenate([np.arange(0, 40), rng.integers(1, 20, n - 40)]))
    cols = [np.sort(rng.choice(n, size=int(L), replace=False)) for L in lengths]
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(lengths)
    colidx = np.concatenate(cols).astype(np.int32)
    vals = rng.uniform(0.5, 1.5, colidx.size).astype(np.float32)
    X = rng.uniform(-1, 1, (n, F)).astype(np.float32)
    X[7], X[31, ::2], X[50, 1::3] = np.inf, -np.inf, np.nan
    d = DeviceCSR(rowptr, colidx, vals, X)
    if ld:
        wide = torch.empty((n - 1) * ld + F, dtype=torch.float32, device="cuda:0").as_strided((n, F), (ld, 1))
        wide.copy_(d.X)
        d.X, d.F = wide, F
    for mode, W in (("full", 0), ("bucket", 9), ("bucket", 13)):
        ref = np.zeros((n, F))
        with np.errstate(invalid="ignore"):
            for r in range(n):
                for p in range(rowptr[r], rowptr[r + 1] if mode == "full" else min(rowptr[r + 1], rowptr[r] + W)):
                    ref[r] += float(vals[p]) * X[colidx[p]].astype(np.float64)
        opts = dict(kernel=2)
        if lanes:
            opts["lanes_per_row"] = lanes
        Y = d.run(W, mode, opts=opts).cpu().numpy()
        for name, pick in (("nan", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
            assert np.array_equal(pick(Y), pick(ref)), f"{name} F={F} ld={ld} {mode} W={W}"
        fine = np.isfinite(ref)
        assert np.abs(Y[fine] - ref[fine]).max() <= 1e-5 * 40      # at most 39 terms of magnitude 1.5


@pytest.mark.parametrize("F,lanes", [(16, 0), (64, 8), (128, 0), (41, 0)])
@pytest.mark.parametrize("n,ld", [(60, 0), (508, 1 << 21), (509, 1 << 21)])
def test_flattened_kernel_strided_rows_and_offsets_up_to_4_gb(es, F, lanes, n, ld):
    """FastRand's strided entries beside absent ones, with infinities in X; 508 rows 8 MiB apart are the largest table that is
    addressed by 32-bit byte offsets (4.26 GB, most of them beyond 2 GiB), one more takes the 64-bit form."""
    import torch
    import oracle
    from gpu_util import DeviceCSR
    rng = np.random.default_rng(F + lanes + n)
    lengths = rng.permutation(np.concatenate([np.arange(0, 40), rng.integers(1, 50, n - 40)]))
    cols = [np.sort(rng.choice(n, size=int(L), replace=False)) for L in lengths]
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(lengths)
    colidx = np.concatenate(cols).astype(np.int32)
    assert (colidx >= 0.95 * n).any()
    vals = rng.uniform(0.5, 1.5, colidx.size).astype(np.float32)
    X = rng.uniform(-1, 1, (n, F)).astype(np.float32)
    X[7], X[31, ::2], X[n - 1, 1::3], X[0, 3] = np.inf, -np.inf, np.nan, np.inf
    d = DeviceCSR(rowptr, colidx, vals, X)
    if ld:
        wide = torch.empty((n - 1) * ld + F, dtype=torch.float32, device="cuda:0").as_strided((n, F), (ld, 1))
        wide.copy_(d.X)
        d.X, d.F = wide, F
    for mode, W, seed in (("full", 0, 0), ("bucket", 9, 0), ("fastrand", 9, 0), ("fastrand", 13, 2 ** 63 + 5)):
        ref = np.zeros((n, F))
        kept = (np.stack([np.arange(rowptr[-1]), np.repeat(np.arange(n), lengths)], axis=1).tolist() if mode == "full" else
                [(q, r) for r, row in enumerate(oracle.kept(rowptr, W, mode, seed)[0].reshape(n, W)) for q in row if q >= 0])
        with np.errstate(invalid="ignore"):
            for q, r in kept:
                ref[r] += float(vals[q]) * X[colidx[q]].astype(np.float64)
        opts = dict(kernel=2, **(dict(lanes_per_row=lanes) if lanes else {}))
        Y = d.run(W, mode, seed, opts=opts).cpu().numpy()
        for name, pick in (("nan", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
            assert np.array_equal(pick(Y), pick(ref)), f"{name} F={F} n={n} {mode} W={W} seed={seed}"
        fine = np.isfinite(ref)
        assert np.abs(Y[fine] - ref[fine]).max() <= 1e-5 * 50      # at most 49 terms of magnitude 1.5


@pytest.mark.parametrize("F,lanes", [(16, 0), (64, 8), (64, 0), (128, 0), (256, 0), (41, 0)])
def test_flattened_kernel_bursts_and_shares(es, F, lanes):
    """The flattened kernel around the sizes a workgroup counts in: bursts of 1536
    and 2048 entries, quarter shares of a burst (a row that ends on, before and
    behind a share's border, one that spans several shares or bursts), runs of
    empty rows longer than a workgroup's 64, and FastRand beyond the width up to
    which its index fits a 24-bit product (28000)."""
    from gpu_util import DeviceCSR, check_against_oracle
    n = 6200
    rng = np.random.default_rng(77 + F + lanes)
    runs = [[384] * 9 + [383, 385, 7, 1], [512] * 9 + [511, 513, 520], [1536, 1535, 1537, 8, 2048, 2047, 2049],
            [5000, 1, 0, 6144, 3], [0] * 130 + [1], [4096] + [0] * 62 + [9], [8] * 192 + [1] * 64]
    lengths = [L for run in runs for L in run]
    cols = [np.sort(rng.choice(n, size=int(L), replace=False)) for L in lengths]
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:len(lengths) + 1] = np.cumsum([len(c) for c in cols])
    rowptr[len(lengths) + 1:] = rowptr[len(lengths)]
    colidx = np.concatenate(cols).astype(np.int32)
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    X = rng.uniform(-1, 1, (n, F)).astype(np.float32)
    d = DeviceCSR(rowptr, colidx, vals, X).with_workspace()
    base = dict(kernel=2, workspace=d.default_ws)
    if lanes:
        base["lanes_per_row"] = lanes
    _say(f"bursts and shares F={F} lanes={lanes}")
    for extra in (dict(long_row_threshold=100000), dict(long_row_threshold=1500), dict(column_partition=1)):
        opts = dict(base, **extra)
        check_against_oracle(d, 0, "full", what=f"full F={F} {extra}", opts=opts)
        for mode, W in (("bucket", 384), ("bucket", 3000), ("fastrand", 384), ("fastrand", 3000)):
            check_against_oracle(d, W, mode, 5, norm="mean", what=f"{mode} W={W} F={F} {extra}", opts=opts)
    m = 29_600                                # two rows beyond the 24-bit width, on both sides of it
    rowptr = np.zeros(m + 1, dtype=np.int32)
    rowptr[1], rowptr[2:] = m, 2 * m - 100
    colidx = np.concatenate([np.arange(m), np.arange(m - 100)]).astype(np.int32)
    d = DeviceCSR(rowptr, colidx, None, rng.uniform(-1, 1, (m, F)).astype(np.float32))
    for W in (27_999, 28_000, 29_500, 29_550):
        for thr in (100000, 1500):
            check_against_oracle(d, W, "fastrand", 3, what=f"wide fastrand W={W} F={F} long rows above {thr}",
                                 opts=dict(kernel=2, long_row_threshold=thr))


@pytest.mark.parametrize("F,lengths", [
    (3, [3900, 1025, 1024, 1023, 513, 512, 511, 257, 256, 255, 65, 64, 0, 1]),
    (16, [3270, 1025, 1024, 1023, 513, 512, 511, 257, 256, 255, 65, 64, 0, 1]), (16, [520] * 20 + [70] * 70),
    (41, [2490, 1300, 1024, 513, 512, 257, 256, 65]), (64, [2048, 1100, 1025, 513, 512, 257, 256, 65, 0]),
    (130, [1340, 1040, 513, 512, 300, 257, 256, 65]), (256, [819, 513, 512, 257, 256, 65]),
    (602, [393, 300, 257, 256, 70, 65])])
def test_long_rows_of_a_small_product(es, F, lengths):
    """Within the bounds on the longest row and on the entries a long row is one
    wave's or one workgroup's (segments of 256 dealt to four waves, partial sums
    added through LDS) and nothing is zeroed first: row lengths around a segment,
    two and four, more rows than waves and workgroups share; the same rows through
    the split-and-atomics form (a larger nnz hint)."""
    import torch
    from gpu_util import DeviceCSR, check_against_oracle, check_Y
    import oracle
    n = 262144 // (F + 64)
    rng = np.random.default_rng(F)
    cols = [np.sort(rng.choice(n, size=L, replace=False)) for L in lengths]
    rowptr = np.zeros(n + 1, dtype=np.int32)
    at = rng.permutation(min(n, 1000))[:len(lengths)]
    counts = np.zeros(n, dtype=np.int64)
    counts[at] = [len(c) for c in cols]
    rowptr[1:] = np.cumsum(counts)
    colidx = np.concatenate([c for _, c in sorted(zip(at, cols), key=lambda t: t[0])]).astype(np.int32)
    assert colidx.size * (F + 64) <= 5 * 262144
    d = DeviceCSR(rowptr, colidx, rng.standard_normal(colidx.size).astype(np.float32),
                  rng.uniform(-1, 1, (n, F)).astype(np.float32))
    for mode, W in (("full", 0), ("bucket", 1100), ("fastrand", 290)):
        for norm in ("none", "mean"):
            check_against_oracle(d, W, mode, 5, norm=norm, what=f"{mode} W={W} F={F} {norm}", opts=dict(long_row_threshold=64))
            Y = torch.full((n, F), float("nan"), device=d.X.device)
            es.es_spmm_ex(d.rowptr, d.colidx, d.vals, d.X, Y, W, mode, 5, norm, dict(long_row_threshold=64), nnz=10_000_000)
            torch.cuda.synchronize()
            ref, den = oracle.spmm(d.h_rowptr, d.h_colidx, d.h_vals, d.h_X, F, W, mode, 5, norm=norm)
            check_Y(Y.cpu().numpy(), ref, den, f"split {mode} W={W} F={F} {norm}")


def test_a_hint_far_below_the_truth_changes_no_result(es):
    """nnz is a hint: with one of 1000 for a row of 2^30 + 1000 entries the library
    takes the small-product form, in which such a row is still one task.  Sixteen
    entries pick the row of ones (on both sides of entry 2^30), the others a row of
    zeros, so the sum is exact."""
    import torch
    n = (1 << 30) + 1000
    rowptr = torch.tensor([0, n, n], dtype=torch.int32, device="cuda")
    colidx = torch.zeros(n, dtype=torch.int32, device="cuda")
    colidx[torch.tensor([0, 63, 255, 256, 1023, 1024, 99_999, (1 << 30) - 1, 1 << 30, (1 << 30) + 1, n - 257, n - 256,
                         n - 3, n - 2, n - 1, 12_345_678], device="cuda")] = 1
    X = torch.tensor([[0.0] * 4, [1.0, 2.0, 3.0, 4.0]], device="cuda")
    for hint in (1000, n):
        _say(f"row of {n} entries, hint {hint}")
        Y = torch.full((2, 4), float("nan"), device="cuda")
        es.es_spmm(rowptr, colidx, None, X, Y, 0, "full", nnz=hint)
        torch.cuda.synchronize()
        assert Y.tolist() == [[16.0, 32.0, 48.0, 64.0], [0.0] * 4], hint
    del colidx
    torch.cuda.empty_cache()


def test_native_marshalling_of_streams_and_integers(es):
    """Explicit streams (torch streams, raw addresses) and NumPy integers are
    marshalled natively and mean what they mean in the Python checks: the native
    call answers 0 and writes the product; what those checks refuse stays refused."""
    import torch
    import oracle
    from gpu_util import check_Y
    n, F = 500, 16
    rowptr, colidx, vals, Xh = _random_graph(n, 9.0, seed=3, F=F)
    rp, ci, va, X = (torch.from_numpy(a).cuda() for a in (rowptr, colidx, vals, Xh))
    t = es.es_spmm_transpose_graph(rp, ci, va)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    m = es.load_marshal()
    Yref, den = oracle.spmm(rowptr, colidx, vals, Xh, F, 4, "fastrand", 9)
    Bref, bden = oracle.spmm_backward(rowptr, colidx, vals, Xh, F, 4, "fastrand", 9)
    for stream in (None, 0, side, side.cuda_stream, torch.cuda.default_stream()):
        for W, seed, f, nnz in ((4, 9, None, None), (np.int64(4), np.uint64(9), np.int32(F), np.int64(colidx.size))):
            what = f"stream {stream!r} {type(W).__name__}"
            Y = torch.full((n, F), float("nan"), device="cuda")
            torch.cuda.synchronize()
            assert m.spmm(rp, ci, va, X, Y, W, "fastrand", seed, np.int8(0), None, f, stream, nnz) == 0, what
            torch.cuda.synchronize()
            check_Y(Y.cpu().numpy(), Yref, den, what)
            assert m.backward(rp, ci, va, X, Y, W, np.int64(2), seed, "none", f, stream, nnz) == 0, what
            torch.cuda.synchronize()
            check_Y(Y.cpu().numpy(), Bref, bden, "backward " + what)
            assert m.pull(rp, t, X, Y, W, "fastrand", seed, "none", f, stream) == 0, what
            torch.cuda.synchronize()
            check_Y(Y.cpu().numpy(), Bref, bden, "pull " + what)
    Y = torch.empty((n, F), device="cuda")
    for bad in (dict(stream="x"), dict(F=16.5), dict(F=F + 1), dict(F=np.int64(F + 1)), dict(nnz=3.0), dict(stream=1.5)):
        args = dict(dict(F=None, stream=None, nnz=None), **bad)
        assert m.spmm(rp, ci, va, X, Y, 4, "bucket", 0, "none", None, args["F"], args["stream"], args["nnz"]) is None, bad
        with pytest.raises((TypeError, ValueError, AttributeError, ctypes.ArgumentError)):
            es.es_spmm(rp, ci, va, X, Y, 4, "bucket", **bad)
    for odd in (dict(W=4.0), dict(W="4"), dict(seed=9.0)):           # what int() takes is still taken
        es.es_spmm(rp, ci, va, X, Y, odd.get("W", 4), "fastrand", odd.get("seed", 9))
        torch.cuda.synchronize()
        check_Y(Y.cpu().numpy(), Yref, den, f"{odd}")


def test_degenerate_inputs(es):
    import torch
    from gpu_util import DeviceCSR, check_against_oracle
    # all rows empty
    n = 130
    rowptr = np.zeros(n + 1, dtype=np.int32)
    colidx = np.zeros(0, dtype=np.int32)
    X = np.ones((n, 8), dtype=np.float32)
    d = DeviceCSR(rowptr, colidx, np.zeros(0, dtype=np.float32), X)
    for mode, W in (("full", 0), ("bucket", 4), ("fastrand", 4)):
        Y = d.run(W, mode)
        assert (Y == 0).all()
    # single row, single entry; unweighted graph (vals == NULL)
    d1 = DeviceCSR(np.array([0, 1], dtype=np.int32), np.array([0], dtype=np.int32), None,
                   np.full((1, 4), 2.5, dtype=np.float32))
    for mode, W in (("full", 0), ("bucket", 1), ("fastrand", 9)):
        assert (d1.run(W, mode).cpu().numpy() == 2.5).all()
    rowptr, colidx, _, X = _random_graph(300, 6.0, seed=3, F=12, unit_vals=True)
    du = DeviceCSR(rowptr, colidx, None, X)
    for mode, W in (("full", 0), ("bucket", 2), ("fastrand", 2)):
        check_against_oracle(du, W, mode, 5, what=f"unit values {mode}")
    # the nnz argument is only a launch-shape hint: any value gives the same result
    import paper_2104_10716_amd as esm
    rowptr, colidx, vals, X = _random_graph(400, 40.0, seed=8, F=32)
    dh = DeviceCSR(rowptr, colidx, vals, X)
    for thr in (0, 16):
        opts = dict(long_row_threshold=thr)
        for mode, W in (("full", 0), ("fastrand", 6), ("fastrand", 30)):
            ref = dh.run(W, mode, 3, opts=opts)
            for hint in (0, 1, 10 ** 9):
                Y = torch.empty_like(ref)
                esm.es_spmm_ex(dh.rowptr, dh.colidx, dh.vals, dh.X, Y, W, mode, 3, "none", opts, nnz=hint)
                torch.cuda.synchronize()
                assert torch.allclose(Y, ref, rtol=1e-4, atol=1e-5), (mode, hint)
            check_against_oracle(dh, W, mode, 3, what=f"nnz hint {mode}", opts=opts)
    # N == 0 is a no-op
    e = torch.empty((0, 4), dtype=torch.float32, device="cuda:0")
    es.es_spmm(torch.zeros(1, dtype=torch.int32, device="cuda:0"),
               torch.zeros(0, dtype=torch.int32, device="cuda:0"), None, e, e.clone(), 4, "bucket")
    # errors surface as exceptions with the status, and leave the output untouched
    with pytest.raises(es.EsSpmmError):
        d.run(0, "bucket")
    Yk = torch.full((du.N, du.F), 7.0, dtype=torch.float32, device="cuda:0")
    for bad in (dict(W=0, mode="fastrand"), dict(W=4, mode=9), dict(W=4, mode="bucket", F=du.F + 1)):
        with pytest.raises((es.EsSpmmError, ValueError)):
            es.es_spmm(du.rowptr, du.colidx, du.vals, du.X, Yk, bad["W"], bad["mode"], F=bad.get("F"))
    with pytest.raises(es.EsSpmmError):
        es.es_spmm_norm(du.rowptr, du.colidx, du.vals, du.X, Yk, 4, "bucket", 0, 99)
    with pytest.raises(es.EsSpmmError):
        es.es_spmm_backward(du.rowptr, du.colidx, du.vals, du.X, Yk, 0, "bucket")
    for bad_opts in (dict(rows_per_wave=3), dict(rows_per_wave=128), dict(lanes_per_row=12),
                     dict(long_row_threshold=-1), dict(column_partition=-2)):
        with pytest.raises(es.EsSpmmError):
            es.es_spmm_ex(du.rowptr, du.colidx, du.vals, du.X, Yk, 4, "bucket", 0, "none", bad_opts)
        with pytest.raises(es.EsSpmmError):
            es.es_spmm_backward_ex(du.rowptr, du.colidx, du.vals, du.X, Yk, 4, "bucket", 0, "none", bad_opts)
    torch.cuda.synchronize()
    assert bool((Yk == 7.0).all())
    # runs on a non-default stream too
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        Y = torch.empty((du.N, du.F), dtype=torch.float32, device="cuda:0")
        es.es_spmm(du.rowptr, du.colidx, du.vals, du.X, Y, 2, "fastrand", 5)
    s.synchronize()
    assert torch.equal(Y, du.run(2, "fastrand", 5))


@pytest.mark.parametrize("norm", ["none", "mean", "rsqrt", "rescale", "inv_degree"])
def test_in_kernel_normalisation(es, norm):
    """es_spmm_norm (Section 6.1): row factor of (n, k) applied in the kernel,
    on ordinary rows, on rows sent through the long-row path, and at full size."""
    from gpu_util import DeviceCSR, check_against_oracle
    for F in (16, 41):
        rowptr, colidx, vals, X = _random_graph(900, 25.0, seed=F, F=F, empty_frac=0.1)
        d = DeviceCSR(rowptr, colidx, vals, X)
        for thr in (0, 9):
            opts = dict(long_row_threshold=thr) if thr else None     # None: the es_spmm_norm entry point
            for mode, W in (("full", 0), ("bucket", 6), ("fastrand", 6), ("fastrand", 20), ("fastrand", 1000)):
                check_against_oracle(d, W, mode, 11, norm=norm, opts=opts,
                                     what=f"norm={norm} {mode} W={W} F={F} thr={thr}")
    w = _workload(2)
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X)
    for mode, W in (("full", 0), ("fastrand", 16), ("bucket", 64)):
        worst = check_against_oracle(d, W, mode, 0, norm=norm, what=f"cfg2 norm={norm} {mode} W={W}")
        _say(f"cfg2 norm={norm} {mode} W={W}: max normalised error {worst:.2e}")
    with pytest.raises(es.EsSpmmError):
        d.run(4, "bucket", norm=7)


@pytest.mark.parametrize("F,ldx", [(3, 3), (16, 16), (41, 41), (64, 68), (100, 128), (256, 256), (520, 520)])
def test_backward_small_graphs(es, F, ldx):
    """es_spmm_backward (transposed sampled product) against the oracle on
    ragged small graphs: every mode, row factor, launch shape and the long-row path."""
    from gpu_util import DeviceCSR, check_backward_against_oracle
    rowptr, colidx, vals, dY = _random_graph(650, 12.0, seed=100 + F, F=F, ldx=ldx)
    d = DeviceCSR(rowptr, colidx, vals, dY, F=F)
    maxdeg = int(np.diff(rowptr).max())
    for rpw in (0, 1, 8):
        for thr in (0, 5):
            opts = dict(rows_per_wave=rpw, long_row_threshold=thr) if (rpw or thr) else None
            for mode, W in (("full", 0), ("bucket", 4), ("fastrand", 4), ("fastrand", maxdeg - 1),
                            ("fastrand", maxdeg + 3)):
                for norm in ("none", "mean", "rescale"):
                    check_backward_against_oracle(d, W, mode, 31, norm, opts=opts,
                                                  what=f"backward F={F} {mode} W={W} {norm} rpw={rpw} thr={thr}")
    du = DeviceCSR(rowptr, colidx, None, dY, F=F)              # unweighted
    check_backward_against_oracle(du, 4, "fastrand", 1, what=f"backward unit values F={F}")


@pytest.mark.parametrize("F,ldx", [(3, 3), (16, 16), (41, 41), (64, 68), (100, 128), (256, 256), (520, 520)])
def test_backward_pull_small_graphs(es, F, ldx):
    """es_spmm_backward_pull (gather over the transposed graph, the sampling rule
    inverted per stored entry) against the oracle's transposed product: every
    mode, width, seed and row factor from ONE transposed graph."""
    import torch
    from gpu_util import DeviceCSR, check_backward_pull_against_oracle
    rowptr, colidx, vals, dY = _random_graph(650, 12.0, seed=100 + F, F=F, ldx=ldx)
    d = DeviceCSR(rowptr, colidx, vals, dY, F=F)
    t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
    torch.cuda.synchronize()
    assert int(t["t_ptr"][-1]) == colidx.size and torch.equal(t["t_end"], t["t_ptr"][1:])
    maxdeg = int(np.diff(rowptr).max())
    for mode, W in (("full", 0), ("bucket", 4), ("fastrand", 1), ("fastrand", 4), ("fastrand", maxdeg - 1),
                    ("fastrand", maxdeg + 3)):
        for seed in (0, 31, 2 ** 63 + 5):
            for norm in ("none", "mean", "rescale"):
                check_backward_pull_against_oracle(d, t, W, mode, seed, norm,
                                                   what=f"pull F={F} {mode} W={W} seed={seed} {norm}")
    du = DeviceCSR(rowptr, colidx, None, dY, F=F)              # unweighted: the structure holds ones
    tu = es.es_spmm_transpose_graph(du.rowptr, du.colidx, None)
    check_backward_pull_against_oracle(du, tu, 4, "fastrand", 1, what=f"pull unit values F={F}")


def test_backward_pull_row_lengths_that_change_the_multiplier(es):
    """Rows of 577, 1154, 577*587 and 2*577*587 entries (multipliers 587 and 593)
    and rows spanning several tiles: the inverse of Equation 2 must pick exactly
    the entries the forward sampler reads."""
    from gpu_util import DeviceCSR, check_backward_pull_against_oracle
    rng = np.random.default_rng(3)
    N = 700_000
    lengths = {0: 577, 5: 1154, 9: 577 * 587, 11: 2 * 577 * 587, 40: 5000, 41: 1, 42: 2, 43: 587, 44: 600}
    lens = np.zeros(N, dtype=np.int64)
    for r, L in lengths.items():
        lens[r] = L
    rowptr = np.zeros(N + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(lens)
    colidx = np.concatenate([np.sort(rng.choice(N, size=L, replace=False)) for L in lengths.values()]).astype(np.int32)
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    dY = rng.uniform(-1, 1, (N, 4)).astype(np.float32)
    d = DeviceCSR(rowptr, colidx, vals, dY)
    t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
    for W in (1, 3, 64, 576, 1000, 70_000):
        for seed in (0, 99):
            check_backward_pull_against_oracle(d, t, W, "fastrand", seed, what=f"pull multipliers W={W} seed={seed}")
    check_backward_pull_against_oracle(d, t, 64, "bucket", 0, what="pull multipliers bucket")


def _pull(es, d, t, dX, W, mode="fastrand", seed=7, norm="none", nnz=None):
    """es_spmm_backward_pull with an nnz of the caller's: a hint, by which the kernel is chosen."""
    import torch
    from paper_2104_10716_amd import binding
    rc = es.load_library().es_spmm_backward_pull(
        d.rowptr.data_ptr(), *(t[k].data_ptr() for k in ("t_ptr", "t_row", "t_idx", "t_slot", "t_vals", "t_pinv", "t_rows")),
        d.X.data_ptr(), dX.data_ptr(), d.N, t["t_row"].numel() if nnz is None else nnz, d.F, d.X.stride(0), dX.stride(0), W,
        binding.MODES[mode], seed, binding.NORMS[norm], torch.cuda.current_stream().cuda_stream or None)
    assert rc == 0


def _kernels(call):
    """Names of this library's kernels that `call` launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return " ".join(e.name for e in p.events() if "es_" in e.name)


@pytest.mark.parametrize("F,W", [(16, 1), (16, 3), (32, 8), (41, 4), (3, 64), (16, 65), (3, 90), (260, 2), (131, 5), (255, 33), (512, 2),
                                 (700, 3), (1030, 1)])
def test_backward_pull_with_rows_bits_in_lds(es, F, W):
    """The pull backward where a rotated FastRand's entries are tested against four bits per row first:
    rows of at most W entries, a little longer ones, windows that wrap, rows far longer than sixteen steps; a row
    count that fills no word and no workgroup, an empty column, and a column longer than several passes; rows of 64 lanes
    that are not aligned, two and four column chunks per lane, a second column block."""
    import torch
    import oracle
    from gpu_util import DeviceCSR, check_Y
    N = 24_003
    rng = np.random.default_rng(F * 1000 + W)
    lens = rng.choice([0, 1, 2, 3, 4, 8, 63, 64, 65, 66, 99, 101, 128, 200, 400, 700, 1500], size=N).astype(np.int64)
    lens[rng.choice(N, 60, replace=False)] = 20_000
    lens[:40] = [W, W + 1, 2 * W, 2 * W + 1, 16 * W] * 8
    rows = np.repeat(np.arange(N), lens)
    cols = rng.integers(1, N, rows.size)                           # column 0 stays empty
    cols[rng.random(rows.size) < 0.0005] = 5                       # a column of some 2000 entries
    key = np.unique(rows * N + cols)
    rowptr = np.zeros(N + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(np.bincount(key // N, minlength=N))
    colidx = (key % N).astype(np.int32)
    kept = np.diff(rowptr)
    in_column = np.bincount(colidx, minlength=N)
    assert (kept <= W).any() and (kept > 16 * W).any() and in_column[0] == 0 and in_column[5] > 1_000
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    dY = rng.uniform(-1, 1, (N, F)).astype(np.float32)
    d = DeviceCSR(rowptr, colidx, vals, dY)
    t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
    a, b = (torch.full((N, F), float("nan"), dtype=torch.float32, device="cuda:0") for _ in range(2))
    hint = 2_000_000_000 if F >= 8 else None                       # the widths below stay with es_pull_kernel
    taken = _kernels(lambda: _pull(es, d, t, a, W, nnz=hint))
    assert ("es_pull_filtered_kernel" in taken) == (F >= 8), taken
    for seed, norm in ((2 ** 63 + 5, "rescale"), (7, "none")):
        a.fill_(float("nan"))
        _pull(es, d, t, a, W, seed=seed, norm=norm, nnz=hint)
        torch.cuda.synchronize()
        ref, den = oracle.spmm_backward(rowptr, colidx, vals, dY, F, W, "fastrand", seed, norm=norm)
        check_Y(a.cpu().numpy(), ref, den, f"bits F={F} W={W} seed={seed} {norm}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _pull(es, d, t, b, W, nnz=hint)
    for _ in range(3):
        b.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(a, b)


@pytest.mark.parametrize("F,ldx,rotated,unrotated", [
    # chunks requested together where columns are short: 64 lanes stream (8) unless the short form has the waves for it
    (16, 16, 4, 4), (41, 41, 4, 4), (127, 127, 4, 4), (128, 128, 4, 4), (131, 131, 4, 4), (256, 256, 4, 8), (256, 257, 4, 4), (301, 301, 4, 8),
    (512, 512, 8, 8), (701, 701, 4, 4), (1000, 1000, 8, 8)])
def test_backward_pull_passes(es, F, ldx, rotated, unrotated):
    """Both forms of the pull's passes, by the mean column (96 entries) and the rows' alignment, against the oracle."""
    import torch
    import oracle
    from gpu_util import DeviceCSR, check_Y
    rowptr, colidx, vals, dY = _random_graph(700, 40.0, seed=F, F=F, ldx=ldx)
    d = DeviceCSR(rowptr, colidx, vals, dY, F=F)
    t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
    dX = torch.empty((d.N, F), dtype=torch.float32, device="cuda:0")
    for mode, seed, norm, short in (("fastrand", 7, "mean", rotated), ("fastrand", 0, "none", unrotated), ("bucket", 7, "none", unrotated),
                                    ("bucket", 0, "mean", 4 if ldx == 256 else unrotated)):      # row factors are looked up too
        ref, den = oracle.spmm_backward(rowptr, colidx, vals, dY, F, 9, mode, seed, norm=norm)
        for nnz, chunks in ((12 * d.N, 8 if F == 301 and short == 8 else 4), (12 * d.N + 1, short), (96 * d.N - 1, short), (96 * d.N, 8)):
            dX.fill_(float("nan"))
            taken = _kernels(lambda: _pull(es, d, t, dX, 9, mode, seed, norm, nnz=nnz))
            assert f", {chunks}>" in taken.split("es_pull_kernel")[1], (F, mode, seed, nnz, taken)
            check_Y(dX.cpu().numpy(), ref, den, f"passes F={F} {mode} seed={seed} nnz={nnz}")


@pytest.mark.parametrize("N", [1, 3, 8, 17, 4_097])
def test_backward_pull_with_rows_bits_in_lds_on_few_rows(es, N):
    import torch
    import oracle
    from gpu_util import DeviceCSR, check_Y
    F, W = 20, 2
    rng = np.random.default_rng(N)
    key = np.unique(np.repeat(np.arange(N), 9) * N + rng.integers(0, N, 9 * N))
    rowptr = np.zeros(N + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(np.bincount(key // N, minlength=N))
    colidx = (key % N).astype(np.int32)
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    dY = rng.uniform(-1, 1, (N, F)).astype(np.float32)
    d = DeviceCSR(rowptr, colidx, vals, dY)
    t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
    dX = torch.full((N, F), float("nan"), dtype=torch.float32, device="cuda:0")
    _pull(es, d, t, dX, W, nnz=2_000_000_000)
    torch.cuda.synchronize()
    check_Y(dX.cpu().numpy(), *oracle.spmm_backward(rowptr, colidx, vals, dY, F, W, "fastrand", 7), f"bits N={N}")


@pytest.mark.parametrize("N,nnz,F,W,mode,seed,filtered", [
    (233_000, 113_000_000, 64, 64, "fastrand", 7, True), (233_000, 113_000_000, 64, 64, "fastrand", 0, False),
    (233_000, 113_000_000, 64, 64, "bucket", 7, False),
    # 50 M entries; fewer were 1.05 to 1.36 times as slow where ids cluster
    (150_000, 50_000_000, 64, 16, "fastrand", 7, True), (150_000, 49_999_999, 64, 16, "fastrand", 7, False),
    (40_000, 12_400_000, 16, 20, "fastrand", 7, False), (100_000, 33_900_000, 32, 16, "fastrand", 7, False),
    (70_000, 28_000_000, 64, 37, "fastrand", 7, True), (70_000, 28_000_000, 64, 38, "fastrand", 7, False),
    (70_000, 27_999_999, 64, 16, "fastrand", 7, False), (69_999, 30_000_000, 64, 16, "fastrand", 7, False),
    # gathered columns: 28 a mean entry above 270, and the mean over 0.11
    (200_000, 60_000_000, 16, 17, "fastrand", 7, True), (200_000, 60_000_000, 16, 18, "fastrand", 7, False),
    (200_000, 56_000_000, 64, 16, "fastrand", 7, False),
    (244_000, 244_000 * 490, 64, 69, "fastrand", 7, True), (244_000, 244_000 * 490, 64, 70, "fastrand", 7, False),
    (244_000, 244_000 * 490, 41, 61, "fastrand", 7, True), (244_000, 244_000 * 490, 41, 62, "fastrand", 7, False),
    (150_000, 70_000_000, 8, 16, "fastrand", 7, True), (150_000, 70_000_000, 7, 16, "fastrand", 7, False),
    # rows whose bits fit
    (245_760, 110_000_000, 32, 16, "fastrand", 7, True), (245_761, 110_000_000, 32, 16, "fastrand", 7, False)])
def test_backward_pull_filter_rule(es, N, nnz, F, W, mode, seed, filtered):
    """Where the entries are tested against the rows' bits: by sizes alone, so an almost empty graph shows it."""
    import torch
    from gpu_util import DeviceCSR
    rowptr = np.zeros(N + 1, dtype=np.int32)
    rowptr[1:] = np.minimum(np.arange(1, N + 1), 100)
    d = DeviceCSR(rowptr, np.arange(100, dtype=np.int32), np.ones(100, dtype=np.float32), np.ones((N, F), dtype=np.float32))
    t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
    dX = torch.full((N, F), float("nan"), dtype=torch.float32, device="cuda:0")
    taken = _kernels(lambda: _pull(es, d, t, dX, W, mode, seed, nnz=nnz))
    assert ("es_pull_filtered_kernel" in taken) == filtered and ("es_pull_kernel" in taken) != filtered, taken
    assert bool((dX[:100] == 1).all()) and not bool(dX[100:].any())


def test_backward_pull_full_size(es):
    """Configs 2 and 3 at full size, every element; pull and atomic scatter agree."""
    import torch
    from gpu_util import DeviceCSR, check_backward_pull_against_oracle
    for cfg, cases in ((2, (("fastrand", 16), ("bucket", 128), ("full", 0))), (3, (("fastrand", 64), ("bucket", 16)))):
        w = _workload(cfg)
        dY = np.random.default_rng(cfg).standard_normal((w.N, w.F)).astype(np.float32)
        d = DeviceCSR(w.rowptr, w.colidx, w.vals, dY)
        t = es.es_spmm_transpose_graph(d.rowptr, d.colidx, d.vals)
        for mode, W in cases:
            worst = check_backward_pull_against_oracle(d, t, W, mode, 0, what=f"cfg{cfg} pull {mode} W={W}")
            _say(f"cfg{cfg} backward pull {mode} W={W}: max normalised error {worst:.2e}")
        a = torch.empty((w.N, w.F), dtype=torch.float32, device="cuda:0")
        b = torch.empty_like(a)
        es.es_spmm_backward_pull(d.rowptr, t, d.X, a, 32, "fastrand", 7, "mean")
        es.es_spmm_backward_pull(d.rowptr, t, d.X, b, 32, "fastrand", 7, "mean")
        assert torch.equal(a, b)                                  # no atomics: bit-reproducible
        es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, b, 32, "fastrand", 7, "mean")
        torch.cuda.synchronize()
        assert torch.allclose(a, b, rtol=1e-3, atol=1e-4)
        del d, t, a, b


def test_backward_full_size(es):
    """Transposed product on configs 2 and 3 at full size, every element
    against the oracle; and the adjoint identity <A_s X, dY> = <X, A_s^T dY>
    between the two HIP entry points."""
    import torch
    from gpu_util import DeviceCSR, check_backward_against_oracle
    for cfg, cases in ((2, (("fastrand", 16), ("bucket", 128), ("full", 0))), (3, (("fastrand", 64), ("bucket", 16)))):
        w = _workload(cfg)
        dY = np.random.default_rng(cfg).standard_normal((w.N, w.F)).astype(np.float32)
        d = DeviceCSR(w.rowptr, w.colidx, w.vals, dY)
        for mode, W in cases:
            worst = check_backward_against_oracle(d, W, mode, 0, what=f"cfg{cfg} backward {mode} W={W}")
            _say(f"cfg{cfg} backward {mode} W={W}: max normalised error {worst:.2e}")
        Xd = torch.from_numpy(w.X).to("cuda:0")
        Y = torch.empty((w.N, w.F), dtype=torch.float32, device="cuda:0")
        dX = torch.empty_like(Y)
        es.es_spmm_norm(d.rowptr, d.colidx, d.vals, Xd, Y, 32, "fastrand", 7, "mean")
        es.es_spmm_backward(d.rowptr, d.colidx, d.vals, d.X, dX, 32, "fastrand", 7, "mean")
        lhs = (Y.double() * d.X.double()).sum().item()
        rhs = (Xd.double() * dX.double()).sum().item()
        scale = (Y.double().abs() * d.X.double().abs()).sum().item()
        assert abs(lhs - rhs) <= 1e-5 * scale, (cfg, lhs, rhs)
        _say(f"cfg{cfg}: adjoint identity holds, |lhs-rhs|/scale = {abs(lhs - rhs) / scale:.2e}")
        del d, Xd, Y, dX


def test_scatter_full_size(es):
    """The atomic scatter, which captured streams, callers without memory and es_spmm_backward_ex
    run where es_spmm_backward takes a workspace: configs 2 and 3 at full size, every element."""
    from gpu_util import DeviceCSR, check_backward_against_oracle
    for cfg, mode, W in ((2, "fastrand", 16), (3, "bucket", 16)):
        w = _workload(cfg)
        assert es.es_spmm_backward_workspace_bytes(w.N, w.nnz, w.F, W, mode) > 0
        dY = np.random.default_rng(cfg).standard_normal((w.N, w.F)).astype(np.float32)
        d = DeviceCSR(w.rowptr, w.colidx, w.vals, dY)
        worst = check_backward_against_oracle(d, W, mode, 0, what=f"cfg{cfg} scatter {mode} W={W}", opts={})
        _say(f"cfg{cfg} scatter {mode} W={W}: max normalised error {worst:.2e}")
        del d


def _oracle_transposed(rowptr, colidx, vals, W, mode, seed):
    """(column, row, value) of every kept entry, sorted by (column, row)."""
    import oracle
    pos, cnt = oracle.kept(rowptr, W, mode, seed)
    rows = np.repeat(np.arange(rowptr.shape[0] - 1), cnt)
    keep = pos[pos >= 0] if pos.shape[1] else np.zeros(0, dtype=np.int32)
    c = colidx[keep].astype(np.int64)
    v = np.ones(keep.size, dtype=np.float32) if vals is None else vals[keep]
    order = np.lexsort((rows, c))
    return c[order], rows[order], v[order]


@pytest.mark.parametrize("n,avg", [(1, 2.0), (700, 9.0), (40_000, 12.0)])
def test_transposed_sampled_graph(es, n, avg):
    """es_spmm_materialize_transposed: the structure holds exactly the oracle's
    kept entries, grouped by column (order inside a group is free), and the
    full product on it equals the oracle's transposed product."""
    import torch
    import oracle
    from gpu_util import DeviceCSR, check_Y
    rowptr, colidx, vals, dY = _random_graph(n, avg, seed=n + 3, F=20, empty_frac=0.2 if n > 1 else 0.0)
    d = DeviceCSR(rowptr, colidx, vals, dY)
    maxdeg = max(1, int(np.diff(rowptr).max()))
    for mode, W in (("bucket", 3), ("fastrand", 3), ("fastrand", maxdeg + 2), ("full", 0)):
        for seed in (0, 5):
            ptr, end, idx, val = es.es_spmm_materialize_transposed(d.rowptr, d.colidx, d.vals, W, mode, seed)
            torch.cuda.synchronize()
            ptr_h, end_h = ptr.cpu().numpy(), end.cpu().numpy()
            ec, er, ev = _oracle_transposed(rowptr, colidx, vals, W, mode, seed)
            total = ec.size
            assert ptr_h[0] == 0 and ptr_h[-1] == total
            assert np.array_equal(np.diff(ptr_h), np.bincount(ec, minlength=n)), (mode, W, seed)
            assert np.array_equal(end_h, ptr_h[1:])
            gc = np.repeat(np.arange(n), np.diff(ptr_h))
            gr = idx.cpu().numpy()[:total].astype(np.int64)
            gv = val.cpu().numpy()[:total]
            order = np.lexsort((gr, gc))
            assert np.array_equal(gr[order], er) and np.array_equal(gv[order], ev), (mode, W, seed)
    for norm in ("none", "mean", "inv_degree"):
        ptr, end, idx, val = es.es_spmm_materialize_transposed(d.rowptr, d.colidx, d.vals, 4, "fastrand", 9, norm)
        total = int(ptr[-1].item())
        dX = torch.full((d.N, d.F), float("nan"), dtype=torch.float32, device="cuda:0")
        es.es_spmm(ptr, idx[:total], val[:total], d.X, dX, 0, "full")
        torch.cuda.synchronize()
        ref, den = oracle.spmm_backward(rowptr, colidx, vals, dY, d.F, 4, "fastrand", 9, norm=norm)
        check_Y(dX.cpu().numpy(), ref, den, f"pull backward n={n} norm={norm}")


def test_hip_graph_capture_and_replay(es):
    """es_spmm only enqueues kernels, so a caller can capture it in a HIP graph.
    Replays (with eager work and synchronisations in between) must reproduce the
    eager result every time, also after the inputs change in place."""
    import torch
    from gpu_util import DeviceCSR, check_against_oracle
    rowptr, colidx, vals, X = _random_graph(3000, 20.0, seed=21, F=64)
    d = DeviceCSR(rowptr, colidx, vals, X)
    long_opts = dict(long_row_threshold=24)        # full mode then uses both kernels
    Yf = torch.zeros((d.N, d.F), dtype=torch.float32, device="cuda:0")
    Ys = torch.zeros_like(Yf)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(2):                         # warm-up outside capture
            es.es_spmm_ex(d.rowptr, d.colidx, d.vals, d.X, Yf, 0, "full", 0, "none", long_opts)
            es.es_spmm(d.rowptr, d.colidx, d.vals, d.X, Ys, 8, "fastrand", 5)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        es.es_spmm_ex(d.rowptr, d.colidx, d.vals, d.X, Yf, 0, "full", 0, "none", long_opts)
        es.es_spmm(d.rowptr, d.colidx, d.vals, d.X, Ys, 8, "fastrand", 5)
    for rep in range(4):
        Yf.fill_(float("nan"))
        Ys.fill_(float("nan"))
        if rep == 2:
            d.X.mul_(-0.5)                          # new input values, same buffers
            d.h_X = d.h_X * np.float32(-0.5)
        g.replay()
        torch.cuda.synchronize()
        eager_s = d.run(8, "fastrand", 5)
        assert torch.equal(Ys, eager_s), f"replay {rep}: sampled result differs from eager"
        eager_f = d.run(0, "full", opts=long_opts)
        assert torch.allclose(Yf, eager_f, rtol=1e-4, atol=1e-5), f"replay {rep}: full result differs"
        import oracle
        Yref, den = oracle.spmm(rowptr, colidx, vals, d.h_X, d.F, 8, "fastrand", 5)
        from gpu_util import check_Y
        check_Y(Ys.cpu().numpy(), Yref, den, f"graph replay {rep}")


def test_hip_graph_capture_of_the_partitioned_product(es):
    """The column-partitioned product on the library's static workspace (one
    cuts kernel and eight phase launches, nothing allocated, nothing but kernels)
    inside a HIP graph, on flattened pieces and on the row form: every replay
    equals the eager result bit for bit and stays inside the oracle's bound."""
    import torch
    import oracle
    from gpu_util import DeviceCSR, check_Y
    rowptr, colidx, vals, X = _random_graph(3000, 60.0, seed=23, F=64)
    d = DeviceCSR(rowptr, colidx, vals, X)
    variants = [dict(column_partition=1, kernel=2, lanes_per_row=8), dict(column_partition=1, kernel=1)]
    outs = [torch.zeros((d.N, d.F), dtype=torch.float32, device="cuda:0") for _ in variants]
    for opts in variants:
        info = es.es_spmm_launch_info(d.N, colidx.size, d.F, 0, "full", opts=opts)
        assert info["column_ranges"] == 8 and info["flattened"] == (opts["kernel"] == 2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for Y, opts in zip(outs, variants):                     # warm-up outside capture
            es.es_spmm_static_ws(d.rowptr, d.colidx, d.vals, d.X, Y, 0, "full", 0, "none", opts)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for Y, opts in zip(outs, variants):
            es.es_spmm_static_ws(d.rowptr, d.colidx, d.vals, d.X, Y, 0, "full", 0, "none", opts)
    for rep in range(3):
        for Y in outs:
            Y.fill_(float("nan"))
        if rep == 1:
            d.X.mul_(2.0)                                       # new input values, same buffers
            d.h_X = d.h_X * np.float32(2.0)
        g.replay()
        torch.cuda.synchronize()
        Yref, den = oracle.spmm(rowptr, colidx, vals, d.h_X, d.F, 0, "full", 0)
        for Y, opts in zip(outs, variants):
            eager = torch.empty_like(Y)
            es.es_spmm_static_ws(d.rowptr, d.colidx, d.vals, d.X, eager, 0, "full", 0, "none", opts)
            torch.cuda.synchronize()
            assert torch.equal(Y, eager), f"replay {rep} {opts}: differs from the eager result"
            check_Y(Y.cpu().numpy(), Yref, den, f"graph replay {rep} {opts}")


def test_validate_csr(es):
    """es_spmm_validate_csr reports exactly the faults planted in a host copy of
    a sound graph (and reads nothing it should not while doing so)."""
    import torch
    rowptr, colidx, _, _ = _random_graph(5000, 12.0, seed=77, F=4, empty_frac=0.1)
    N = rowptr.shape[0] - 1
    maxdeg = int(np.diff(rowptr).max())

    def report(rp, ci):
        out = es.es_spmm_validate_csr(torch.from_numpy(rp).to("cuda:0"), torch.from_numpy(ci).to("cuda:0"))
        torch.cuda.synchronize()
        return out.cpu().numpy().tolist()

    assert report(rowptr, colidx) == [0, 0, 0, maxdeg]
    w = _workload(2)
    assert report(w.rowptr, w.colidx) == [0, 0, 0, w.max_degree]
    long_rows = np.nonzero(np.diff(rowptr) >= 3)[0]
    # column ids out of range, in three rows
    ci = colidx.copy()
    for r, bad in zip(long_rows[:3], (-1, N, 2 ** 31 - 1)):
        ci[rowptr[r] + 1] = bad
    rep = report(rowptr, ci)
    assert rep[0] == 0 and rep[1] == 3 and rep[3] == maxdeg
    # unsorted rows (swap two entries): legal, counted
    ci = colidx.copy()
    for r in long_rows[:5]:
        ci[[rowptr[r], rowptr[r] + 1]] = ci[[rowptr[r] + 1, rowptr[r]]]
    assert report(rowptr, ci) == [0, 0, 5, maxdeg]
    # row pointers: one decreasing pair (its two neighbours become faulty pairs), a wrong end, a wrong start
    rp = rowptr.copy()
    rp[100] = rp[101] + 5
    rep = report(rp, colidx)
    assert rep[0] >= 1 and rep[1] == 0
    rp = rowptr.copy()
    rp[-1] += 7                                   # points past the arrays: that row must not be read
    rep = report(rp, colidx)
    assert rep[0] == 2                            # rowptr[N] != nnz, and the last pair exceeds nnz
    rp = rowptr.copy()
    rp[0] = 1
    assert report(rp, colidx)[0] >= 1
    # empty graph
    assert report(np.zeros(4, dtype=np.int32), np.zeros(0, dtype=np.int32)) == [0, 0, 0, 0]


def test_concurrent_streams(es):
    """Calls on two streams at once (different graphs, interleaved launches,
    DIFFERENT launch options on each stream) give what the same calls give one
    after the other: options travel with the call, the library keeps no state
    and every kernel works only on its arguments."""
    import torch
    from gpu_util import DeviceCSR
    ga = DeviceCSR(*_random_graph(20_000, 30.0, seed=51, F=64))
    gb = DeviceCSR(*_random_graph(15_000, 8.0, seed=52, F=128))
    oa = dict(rows_per_wave=1, long_row_threshold=20)            # stream 1: wave per row, long-row path on
    ob = dict(rows_per_wave=8, lanes_per_row=8)                  # stream 2: 8 rows per wave, 32-column slices
    cases = [(ga, 16, "fastrand", 4, oa), (gb, 0, "full", 0, ob), (ga, 0, "full", 0, oa), (gb, 5, "bucket", 0, ob),
             (ga, 100, "fastrand", 9, oa), (gb, 64, "fastrand", 2, ob)]
    serial = [d.run(W, mode, seed, opts=o) for d, W, mode, seed, o in cases]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = [torch.full((d.N, d.F), float("nan"), dtype=torch.float32, device="cuda:0") for d, *_ in cases]
    torch.cuda.synchronize()
    for rep in range(3):
        for i, (d, W, mode, seed, o) in enumerate(cases):
            with torch.cuda.stream(s1 if i % 2 == 0 else s2):
                es.es_spmm_ex(d.rowptr, d.colidx, d.vals, d.X, outs[i], W, mode, seed, "none", o)
    s1.synchronize()
    s2.synchronize()
    for i, (d, W, mode, seed, o) in enumerate(cases):
        atomic_rows = mode == "full" or (o is oa and W > 20)     # long-row part: summation order is free
        if atomic_rows:
            assert torch.allclose(outs[i], serial[i], rtol=1e-4, atol=1e-5), i
        else:
            assert torch.equal(outs[i], serial[i]), i
    # the launch shape each stream asked for is the one its calls got
    ia = es.es_spmm_launch_info(ga.N, ga.h_colidx.size, 64, 16, "fastrand", opts=oa)
    ib = es.es_spmm_launch_info(gb.N, gb.h_colidx.size, 128, 5, "bucket", opts=ob)
    assert ia["rows_per_wave"] == 1 and ia["long_row_threshold"] == 20
    assert ib["rows_per_wave"] == 8 and ib["lanes_per_row"] == 8 and ib["grid_y"] == 4


def _one_row_graph(n):
    """rowptr of a 3-row matrix whose middle row has n entries (only the row
    pointers matter to the sampler export)."""
    return np.array([0, 5, 5 + n, 5 + n + 7], dtype=np.int32)


@pytest.mark.parametrize("n,W", [(338_699, 3), (338_699, 64), (200_848_507, 3), (200_848_507, 64),
                                 (2 * 338_699, 64), (577 * 1000, 700)])
def test_sampler_multiplier_fallbacks(es, n, W):
    """Row lengths divisible by 577*587 (multiplier 593) and by 577*587*593
    (multiplier 599): the device sampler's picks equal the oracle's, seeded and
    unseeded, on every lane schedule (Equation 2 with the distinctness reading)."""
    import torch
    import oracle
    rowptr = _one_row_graph(n)
    P = oracle.multiplier(n)
    assert P == (599 if n % (577 * 587 * 593) == 0 else 593 if n % (577 * 587) == 0 else 587)
    drp = torch.from_numpy(rowptr).to("cuda:0")
    for seed in (0, 0xDEADBEEFCAFE):
        opos, ocnt = oracle.kept(rowptr, W, "fastrand", seed)
        assert np.unique(opos[1]).size == W
        for rpw in (0, 1, 4, 64, -1):
            pos, cnt = es.es_spmm_sample_edges(drp, W, "fastrand", seed, rpw)
            torch.cuda.synchronize()
            assert np.array_equal(cnt.cpu().numpy(), ocnt), (n, W, seed, rpw)
            assert np.array_equal(pos.cpu().numpy(), opos), (n, W, seed, rpw)
    _say(f"sampler n={n} (multiplier {P}) W={W}: picks identical to the oracle")


@pytest.mark.parametrize("n", [200_000, 338_699 * 2, 1_000_003])
def test_sampler_slots_above_65535(es, n):
    """W = 70 000 on a row longer than W: slots >= 65 536 take the 64-bit start
    index in the device sampler (tile refills for rows_per_wave >= 0, segment
    restarts for the long-row schedule)."""
    import torch
    import oracle
    W = 70_000
    rowptr = _one_row_graph(n)
    drp = torch.from_numpy(rowptr).to("cuda:0")
    for seed in (0, 991):
        opos, ocnt = oracle.kept(rowptr, W, "fastrand", seed)
        for rpw in (0, -1, 2):
            pos, cnt = es.es_spmm_sample_edges(drp, W, "fastrand", seed, rpw)
            torch.cuda.synchronize()
            assert np.array_equal(cnt.cpu().numpy(), ocnt), (n, seed, rpw)
            got = pos.cpu().numpy()
            assert np.array_equal(got, opos), (n, seed, rpw, int(np.argmax((got != opos).any(axis=0))))
        opos_b, _ = oracle.kept(rowptr, W, "bucket", seed)
        pos, _ = es.es_spmm_sample_edges(drp, W, "bucket", seed, -1)
        assert np.array_equal(pos.cpu().numpy(), opos_b)
    _say(f"sampler n={n} W={W}: slots up to {W - 1} identical to the oracle")


def test_fused_kernel_on_a_very_long_row(es):
    """One es_spmm call with a row of 400 000 entries and W = 70 000: the fused
    kernel's own walk (tile refills past slot 65 536 with a wave per row; 256-slot
    segment restarts on the long-row path) against the oracle, every element."""
    from gpu_util import DeviceCSR, check_against_oracle
    rng = np.random.default_rng(17)
    N = 450_000
    big = np.sort(rng.choice(N, size=400_000, replace=False)).astype(np.int32)
    mid = np.sort(rng.choice(N, size=338_699, replace=False)).astype(np.int32)    # multiplier 593
    small = [np.sort(rng.choice(N, size=L, replace=False)).astype(np.int32) for L in (3, 0, 70_001, 65_537)]
    lists = [small[0], big, small[1], mid, small[2], small[3]]
    rowptr = np.zeros(N + 1, dtype=np.int32)
    lens = np.zeros(N, dtype=np.int64)
    where = [0, 7, 8, 100, 449_998, 449_999]
    for r, l in zip(where, lists):
        lens[r] = l.size
    rowptr[1:] = np.cumsum(lens)
    colidx = np.concatenate(lists)
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    X = rng.uniform(-1, 1, (N, 8)).astype(np.float32)
    d = DeviceCSR(rowptr, colidx, vals, X)
    rows = np.array(where, dtype=np.int64)
    for W in (70_000, 65_536, 3):
        for seed in (0, 5):
            for opts in (dict(rows_per_wave=1, long_row_threshold=2 ** 30), dict(long_row_threshold=1000), None):
                worst = check_against_oracle(d, W, "fastrand", seed, rows=rows, opts=opts,
                                             what=f"very long row W={W} seed={seed} opts={opts}")
    Y = d.run(70_000, "fastrand", 5).cpu().numpy()
    assert np.isfinite(Y).all() and (Y[1:7] == 0).all()          # the empty rows in between are written
    _say(f"fused kernel, row of 400 000 entries at W=70 000: within the bound (worst {worst:.2e})")


def test_determinism_across_launches(es):
    """Same inputs, same launch shape: bit-identical Y and edge lists (the
    sampler is static for a given seed, Section 6.2).  Full mode is
    bit-reproducible on every row below the long-row threshold; longer rows
    are summed through atomic adds and only need to agree within the bound."""
    import torch
    from gpu_util import DeviceCSR
    w = _workload(2)
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X)
    for mode in ("bucket", "fastrand"):
        a = d.run(32, mode, 9)
        b = d.run(32, mode, 9)
        assert torch.equal(a, b)
    a = d.run(0, "full")
    b = d.run(0, "full")
    short = torch.from_numpy(np.diff(w.rowptr) <= 64).to(a.device)      # 64: lowest threshold the host picks
    assert torch.equal(a[short], b[short])
    assert torch.allclose(a, b, rtol=1e-4, atol=1e-5)
    p1, c1 = d.edges(32, "fastrand", 9)
    p2, c2 = d.edges(32, "fastrand", 9)
    assert torch.equal(p1, p2) and torch.equal(c1, c2)
    p0, _ = d.edges(32, "fastrand", 0)
    assert not torch.equal(p0, p1)


def _oracle_sampled_csr(rowptr, colidx, vals, W, mode, seed):
    """Sampled graph as CSR, built on the host from the oracle's kept lists."""
    import oracle
    pos, cnt = oracle.kept(rowptr, W, mode, seed)
    out_rowptr = np.zeros(rowptr.shape[0], dtype=np.int64)
    out_rowptr[1:] = np.cumsum(cnt)
    if pos.shape[1]:
        keep = pos[pos >= 0]                       # row-major: row by row, slot order
    else:
        keep = np.zeros(0, dtype=np.int32)
    v = np.ones(keep.size, dtype=np.float32) if vals is None else vals[keep]
    return out_rowptr.astype(np.int32), colidx[keep], v


@pytest.mark.parametrize("n,avg", [(1, 3.0), (700, 9.0), (5000, 30.0)])
def test_materialized_sampled_graph(es, n, avg):
    """es_spmm_materialize (pre-sampled graph of Section 5.6): the CSR it writes
    equals the oracle's kept lists bit for bit, and the full product on it
    equals the fused sampled product."""
    import torch
    from gpu_util import DeviceCSR, check_Y
    import oracle
    rowptr, colidx, vals, X = _random_graph(n, avg, seed=n, F=24, empty_frac=0.2 if n > 1 else 0.0)
    d = DeviceCSR(rowptr, colidx, vals, X)
    maxdeg = max(1, int(np.diff(rowptr).max()))
    for mode in ("bucket", "fastrand", "full"):
        for W in (1, 5, maxdeg + 1):
            for seed in (0, 99):
                orp, oci, ova = es.es_spmm_materialize(d.rowptr, d.colidx, d.vals, W, mode, seed)
                torch.cuda.synchronize()
                erp, eci, eva = _oracle_sampled_csr(rowptr, colidx, vals, W, mode, seed)
                kept = int(erp[-1])
                assert np.array_equal(orp.cpu().numpy(), erp), (mode, W, seed)
                assert np.array_equal(oci.cpu().numpy()[:kept], eci), (mode, W, seed)
                assert np.array_equal(ova.cpu().numpy()[:kept], eva), (mode, W, seed)
                Y = torch.full((d.N, d.F), float("nan"), dtype=torch.float32, device="cuda:0")
                es.es_spmm(orp, oci[:kept], ova[:kept], d.X, Y, 0, "full")
                torch.cuda.synchronize()
                Yref, den = oracle.spmm(rowptr, colidx, vals, X, d.F, W, mode, seed)
                check_Y(Y.cpu().numpy(), Yref, den, f"full product on materialised {mode} W={W}")
    # unweighted input writes ones
    orp, oci, ova = es.es_spmm_materialize(d.rowptr, d.colidx, None, 3, "fastrand", 1)
    torch.cuda.synchronize()
    assert (ova.cpu().numpy()[:int(orp[-1])] == 1.0).all()


def test_materialized_row_pointers_many_blocks(es):
    """Row-pointer scan across many 1024-row blocks (config 2, 170 k rows)."""
    import torch
    w = _workload(2)
    from gpu_util import DeviceCSR
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X)
    for mode, W in (("fastrand", 16), ("bucket", 128), ("full", 0)):
        orp, oci, ova = es.es_spmm_materialize(d.rowptr, d.colidx, d.vals, W, mode, 0)
        torch.cuda.synchronize()
        erp, eci, eva = _oracle_sampled_csr(w.rowptr, w.colidx, w.vals, W, mode, 0)
        kept = int(erp[-1])
        assert np.array_equal(orp.cpu().numpy(), erp)
        assert np.array_equal(oci.cpu().numpy()[:kept], eci)
        assert np.array_equal(ova.cpu().numpy()[:kept], eva)


# --------------------------------------------------------------------------
# the benchmark configurations at full size
# --------------------------------------------------------------------------
def test_config1_tiny_gcn(es):
    from gpu_util import DeviceCSR, check_against_oracle, check_edges
    w = _workload(1)
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X)
    check_against_oracle(d, 0, "full", what="cfg1 full")
    for W in w.Ws:
        for mode in ("bucket", "fastrand"):
            worst = check_against_oracle(d, W, mode, 0, what=f"cfg1 {mode} W={W}")
            check_edges(d, W, mode, 0)
            _say(f"cfg1 {mode} W={W}: max normalised error {worst:.2e}")


def test_config2_citation_like_full_size(es):
    from gpu_util import DeviceCSR, check_against_oracle, check_edges
    w = _workload(2)
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X)
    worst = check_against_oracle(d, 0, "full", what="cfg2 full")
    _say(f"cfg2 full: max normalised error {worst:.2e}")
    for W in w.Ws:
        for mode in ("bucket", "fastrand"):
            worst = check_against_oracle(d, W, mode, 0, what=f"cfg2 {mode} W={W}")
            check_edges(d, W, mode, 0)
            _say(f"cfg2 {mode} W={W}: max normalised error {worst:.2e}")


def _cfg3_device():
    """Config 3 on the device, calls routed through es_spmm_ws as in bench.py (the
    exact product then runs column-partitioned)."""
    from gpu_util import DeviceCSR
    w = _workload(3)
    return w, DeviceCSR(w.rowptr, w.colidx, w.vals, w.X).with_workspace()


def test_config3_social_like_full_product(es):
    """Config 3 (113 M entries, rows up to 20 k): EVERY element of the exact
    product against the oracle, in row blocks -- through es_spmm_ws (column-
    partitioned) and through plain es_spmm (rows up to 20 k on the long-row path)."""
    from gpu_util import check_every_element
    w, d = _cfg3_device()
    worst = check_every_element(d, 0, "full", what="cfg3 full")
    _say(f"cfg3 full (es_spmm_ws): max normalised error {worst:.2e} over all {w.N} x {w.F} elements")
    d.default_ws = None
    worst = check_every_element(d, 0, "full", what="cfg3 full, no workspace")
    _say(f"cfg3 full (es_spmm): max normalised error {worst:.2e} over all {w.N} x {w.F} elements")


@pytest.mark.parametrize("mode", ["bucket", "fastrand"])
def test_config3_social_like_every_width(es, mode):
    """Config 3, every W of the sweep: every element of Y against the oracle."""
    from gpu_util import check_every_element
    w, d = _cfg3_device()
    for W in w.Ws:
        worst = check_every_element(d, W, mode, 0, what=f"cfg3 {mode} W={W}")
        _say(f"cfg3 {mode} W={W}: max normalised error {worst:.2e} over all {w.N} x {w.F} elements")


@pytest.mark.parametrize("cfg", [2, 3, 4])
def test_flattened_kernel_full_size(es, cfg):
    """The flattened kernel forced on at full size: every element of Y against the
    oracle for the smallest and largest W of the sweep and the exact product
    (config 3: column-partitioned as well)."""
    from gpu_util import DeviceCSR, check_every_element
    w = _workload(cfg)
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X).with_workspace()
    cases = [("bucket", w.Ws[0]), ("fastrand", w.Ws[0]), ("fastrand", w.Ws[-1]), ("full", 0)]
    for mode, W in cases:
        opts = dict(workspace=d.default_ws, kernel=2)
        worst = check_every_element(d, W, mode, 0, what=f"cfg{cfg} flattened {mode} W={W}", opts=opts)
        _say(f"cfg{cfg} flattened {mode} W={W}: max normalised error {worst:.2e}")
    if cfg == 3:
        worst = check_every_element(d, 0, "full", what="cfg3 flattened, not partitioned",
                                    opts=dict(workspace=d.default_ws, kernel=2, column_partition=-1))
        _say(f"cfg3 flattened exact product without column ranges: max normalised error {worst:.2e}")


@pytest.mark.parametrize("cfg", [3, 4])
def test_row_kernel_forced_full_size(es, cfg):
    """The row kernel forced on where the library would by itself run the
    flattened one (config 4 at every width, config 3's partitioned exact product):
    every element of Y against the oracle."""
    from gpu_util import DeviceCSR, check_every_element
    w = _workload(cfg)
    d = DeviceCSR(w.rowptr, w.colidx, w.vals, w.X).with_workspace()
    assert es.es_spmm_launch_info(w.N, w.nnz, w.F, 0, "full")["flattened"] == 1
    assert es.es_spmm_launch_info(w.N, w.nnz, w.F, 0, "full", opts=dict(kernel=1))["flattened"] == 0
    cases = [("full", 0)] if cfg == 3 else [("fastrand", w.Ws[0]), ("bucket", w.Ws[-1]), ("full", 0)]
    for mode, W in cases:
        worst = check_every_element(d, W, mode, 0, what=f"cfg{cfg} row kernel {mode} W={W}",
                                    opts=dict(workspace=d.default_ws, kernel=1))
        _say(f"cfg{cfg} row kernel {mode} W={W}: max normalised error {worst:.2e}")


def test_column_ranges_of_rows_that_tile_no_line(es):
    """What the library chooses above 125 k rows where F is no multiple of 32: column ranges on the
    flattened kernel, one slice (F = 20, 28), a second of few columns (68) and 64-column slices (100, 124)."""
    from gpu_util import DeviceCSR, check_every_element
    N = 126_001
    rowptr, colidx, vals, X = _random_graph(N, 138.0, seed=3, F=124, empty_frac=0.02)
    for F in (20, 28, 68, 100, 124):
        info = es.es_spmm_launch_info(N, colidx.size, F, 0, "full", ldx=124)
        assert info["column_ranges"] == 8 and info["flattened"] == 1 and info["lanes_per_row"] == (8 if F < 64 else 16), (F, info)
        d = DeviceCSR(rowptr, colidx, vals, X, F=F).with_workspace()
        worst = check_every_element(d, 0, "full", what=f"ranges F={F}", norm="mean")
        _say(f"column ranges on the flattened kernel, F={F}: max normalised error {worst:.2e}")
        del d


def test_config3_column_partitioned(es):
    """Config 3 through es_spmm_ws (the library itself chooses the column-
    partitioned product here): every element against the oracle, and the result
    is bit-identical from launch to launch."""
    import torch
    from gpu_util import check_every_element
    w, d = _cfg3_device()
    info = es.es_spmm_launch_info(w.N, w.nnz, w.F, 0, "full")
    assert info["column_ranges"] == 8, info
    ws = torch.empty(es.es_spmm_workspace_bytes(w.N) // 4, dtype=torch.int32, device="cuda:0")
    for mode, W in (("full", 0), ("fastrand", 256), ("fastrand", 2304)):
        opts = dict(workspace=ws, column_partition=0 if mode == "full" else 1)   # FastRand: only on request
        worst = check_every_element(d, W, mode, 0, what=f"cfg3 partitioned {mode} W={W}", opts=opts)
        _say(f"cfg3 es_spmm_ws {mode} W={W}: max normalised error {worst:.2e} over all {w.N} x {w.F} elements")
    a = d.run(0, "full", opts=dict(workspace=ws))
    b = d.run(0, "full", opts=dict(workspace=ws))
    assert torch.equal(a, b)


def test_config3_social_like_edge_lists(es):
    """Config 3: sampled edge lists of every row, bit-exact (smallest and
    largest W, a 60-bit seed, the long-row sampler schedule)."""
    from gpu_util import check_edges, check_every_element
    w, d = _cfg3_device()
    for W in (16, 256):
        for mode in ("bucket", "fastrand"):
            check_edges(d, W, mode, 0)
            _say(f"cfg3 {mode} W={W}: edge lists identical")
    check_edges(d, 64, "fastrand", 0xC0FFEE123456789)
    check_edges(d, 64, "fastrand", 3, rows_per_wave=-1)
    check_edges(d, 300, "fastrand", 3, rows_per_wave=-1)
    worst = check_every_element(d, 64, "fastrand", 0xC0FFEE123456789, what="cfg3 fastrand W=64 seeded")
    _say(f"cfg3 fastrand W=64 with a 60-bit seed: edge lists identical, max normalised error {worst:.2e}")


@pytest.mark.parametrize("W", [1792, 2304])
def test_config3_widths_of_the_paper_densest_graph(es, W):
    """The widths the paper needs for Bucket on its densest graph (S = 1792,
    2304): several LDS tiles per row and rows above the long-row threshold;
    every element against the oracle."""
    from gpu_util import check_every_element
    w, d = _cfg3_device()
    for mode in ("bucket", "fastrand"):
        worst = check_every_element(d, W, mode, 0, what=f"cfg3 {mode} W={W}")
        _say(f"cfg3 {mode} W={W}: max normalised error {worst:.2e} over all {w.N} x {w.F} elements")


@pytest.mark.parametrize("cfg", [3, 4])
def test_full_size_every_row_counts_its_kept_entries(es, cfg):
    """A property that holds at any size and covers EVERY row of the big
    graphs: with unit values and X = 1 each output equals the number of kept
    entries min(deg, W) (Section 4.2), exactly -- small integers are exact in
    fp32 whatever the summation order."""
    import torch
    w = _workload(cfg)
    dev = "cuda:0"
    rowptr = torch.from_numpy(w.rowptr).to(dev)
    colidx = torch.from_numpy(w.colidx).to(dev)
    F = 8
    X = torch.ones((w.N, F), dtype=torch.float32, device=dev)
    Y = torch.empty((w.N, F), dtype=torch.float32, device=dev)
    deg = torch.from_numpy(np.diff(w.rowptr).astype(np.float32)).to(dev)
    for mode, W in (("full", 0), ("bucket", 16), ("fastrand", 16), ("fastrand", 256), ("bucket", 2304)):
        Y.fill_(float("nan"))
        es.es_spmm(rowptr, colidx, None, X, Y, W, mode, 0)
        torch.cuda.synchronize()
        expect = deg if mode == "full" else torch.clamp(deg, max=float(W))
        assert torch.equal(Y, expect[:, None].expand(-1, F)), f"cfg{cfg} {mode} W={W}"
        _say(f"cfg{cfg} {mode} W={W}: all {w.N} rows count their kept entries exactly")
    # X[j] = j (exact in fp32 below 2^24) with a single column: FastRand must
    # pick exactly the oracle's columns; compare the exact integer sums of the
    # column ids on every row whose sum stays below 2^24
    if w.N < 2 ** 24:
        import oracle
        Xid = torch.arange(w.N, dtype=torch.float32, device=dev).reshape(-1, 1).repeat(1, 4).contiguous()
        Y4 = torch.empty((w.N, 4), dtype=torch.float32, device=dev)
        W = 4
        es.es_spmm(rowptr, colidx, None, Xid, Y4, W, "fastrand", 0)
        torch.cuda.synchronize()
        pos, cnt = oracle.kept(w.rowptr, W, "fastrand", 0)
        cols = np.where(pos >= 0, w.colidx[np.maximum(pos, 0)], 0).astype(np.int64)
        sums = cols.sum(axis=1)
        ok = sums < 2 ** 24
        # partial sums of non-negative integers below 2^24 are exact in any order
        got = Y4[:, 0].cpu().numpy().astype(np.int64)
        assert np.array_equal(got[ok], sums[ok]), f"cfg{cfg}: column-id sums differ"
        _say(f"cfg{cfg} fastrand W=4: column-id sums exact on {int(ok.sum())} of {w.N} rows")


def test_maximum_sizes_int32_index_range(es):
    """nnz just below 2^31 (the int32 CSR limit) and N*W just below 2^31 for the
    sampler export: 4 Mi rows of 511 entries.  The graph is drawn on the device
    (torch, seeded) because 2.1 G entries are too many to push through the host;
    checks: every row's exact kept count, and the oracle on sampled rows whose
    entries are copied back."""
    import torch
    import oracle
    from gpu_util import check_Y
    dev = "cuda:0"
    N, deg, F = 1 << 22, 511, 4
    nnz = N * deg
    assert nnz < 2 ** 31 and nnz > 2 ** 31 - 2 ** 23
    g = torch.Generator(device=dev)
    g.manual_seed(1234)
    colidx = torch.randint(0, N, (nnz,), dtype=torch.int32, device=dev, generator=g)
    rowptr = (torch.arange(N + 1, dtype=torch.int64, device=dev) * deg).to(torch.int32)
    ones = torch.ones((N, F), dtype=torch.float32, device=dev)
    Y = torch.empty((N, F), dtype=torch.float32, device=dev)
    for mode, W in (("fastrand", 16), ("bucket", 500), ("full", 0)):
        Y.fill_(float("nan"))
        es.es_spmm(rowptr, colidx, None, ones, Y, W, mode, 0)
        torch.cuda.synchronize()
        expect = float(deg if mode == "full" else min(deg, W))
        assert bool((Y == expect).all()), f"max size {mode} W={W}"
        _say(f"max size nnz={nnz}: {mode} W={W} counts exact on all {N} rows")
    # oracle on sampled rows (last rows included: their entries sit at the top of the index range)
    rows = np.unique(np.concatenate([np.random.default_rng(0).integers(0, N, 300),
                                     [0, N - 1, N - 2, N // 2]])).astype(np.int64)
    sub_cols = np.stack([colidx[r * deg:(r + 1) * deg].cpu().numpy() for r in rows])
    sub_rowptr = (np.arange(rows.size + 1, dtype=np.int64) * deg).astype(np.int32)
    Xh = np.random.default_rng(1).uniform(-1, 1, (N, F)).astype(np.float32)
    X = torch.from_numpy(Xh).to(dev)
    for mode, W in (("fastrand", 16), ("fastrand", 500), ("full", 0)):
        es.es_spmm(rowptr, colidx, None, X, Y, W, mode, 0)
        torch.cuda.synchronize()
        Yref, den = oracle.spmm(sub_rowptr, sub_cols.reshape(-1), None, Xh, F, W, mode, 0)
        check_Y(Y.cpu().numpy()[rows], Yref, den, f"max size {mode} W={W}")
    del ones, X
    # sampler export with N*W just below 2^31 (W = 510 < 511 entries per row, so FastRand samples)
    W = 511
    assert N * W < 2 ** 31
    pos, cnt = es.es_spmm_sample_edges(rowptr, W - 1, "fastrand", 0)
    torch.cuda.synchronize()
    assert bool((cnt == W - 1).all())
    opos, ocnt = oracle.kept(sub_rowptr, W - 1, "fastrand", 0)
    got = pos[torch.from_numpy(rows).to(dev)].cpu().numpy().astype(np.int64) - (rows * deg)[:, None]
    assert np.array_equal(got, opos.astype(np.int64) - sub_rowptr[:-1, None].astype(np.int64))
    _say("max size: sampler export matches the oracle on sampled rows")
    del pos, cnt, colidx, rowptr, Y
    torch.cuda.empty_cache()


def _gcn_first_stage_input():
    from workloads import gcn_operands
    g = _workload(3)
    X0, W1, W2 = gcn_operands(g.N)
    Z1 = (X0 @ W1).astype(np.float32)                           # [N x 256]
    return g, Z1, W2


def test_config5_first_stage_F256(es):
    """F = 256 stage of the 2-layer GCN forward (layer equation of Section 2.1:
    GEMM first, then SpMM) on the config-3 graph: every element of Y against
    the oracle for W = 64 (both strategies) and the exact product."""
    from gpu_util import DeviceCSR, check_every_element
    g, Z1, _ = _gcn_first_stage_input()
    d = DeviceCSR(g.rowptr, g.colidx, g.vals, Z1).with_workspace()
    assert es.es_spmm_launch_info(g.N, g.nnz, 256, 0, "full")["column_ranges"] == 8
    for mode, W in (("bucket", 64), ("fastrand", 64), ("full", 0)):
        worst = check_every_element(d, W, mode, 0, what=f"cfg5 F=256 {mode}")
        _say(f"cfg5 F=256 {mode} W={W}: max normalised error {worst:.2e} over all {g.N} x 256 elements")


def test_config5_second_stage_F41(es):
    """F = 41 stage (row stride 41).  The dense products are formed on the host
    from seeded inputs and the ORACLE's first-stage output, so no oracle input
    comes from the HIP path.  Every element against the oracle."""
    import oracle
    from gpu_util import DeviceCSR, check_every_element
    g, Z1, W2 = _gcn_first_stage_input()
    H1, _ = oracle.spmm(g.rowptr, g.colidx, g.vals, Z1, 256, 64, "fastrand", 0, want_denom=False)
    Z2 = (np.maximum(H1, 0.0).astype(np.float32) @ W2).astype(np.float32)   # [N x 41]
    del H1, Z1
    d = DeviceCSR(g.rowptr, g.colidx, g.vals, Z2).with_workspace()
    for mode, W in (("bucket", 64), ("fastrand", 64), ("full", 0)):
        worst = check_every_element(d, W, mode, 0, what=f"cfg5 F=41 {mode}")
        _say(f"cfg5 F=41 {mode} W={W}: max normalised error {worst:.2e} over all {g.N} x 41 elements")
    # and the exact product without a workspace (the unpartitioned kernel on 164-byte rows)
    d.default_ws = None
    worst = check_every_element(d, 0, "full", 0, what="cfg5 F=41 full, no workspace")
    _say(f"cfg5 F=41 full without a workspace: max normalised error {worst:.2e}")


def _cfg4_device():
    from gpu_util import DeviceCSR
    w = _workload(4)
    return w, DeviceCSR(w.rowptr, w.colidx, w.vals, w.X).with_workspace()


def test_config4_copurchase_like_full_product(es):
    """Config 4 (N = 2.45 M, 120 M entries, F = 128): every element of the
    exact product against the oracle, in row blocks."""
    from gpu_util import check_every_element
    w, d = _cfg4_device()
    worst = check_every_element(d, 0, "full", what="cfg4 full")
    _say(f"cfg4 full: max normalised error {worst:.2e} over all {w.N} x {w.F} elements")


@pytest.mark.parametrize("mode", ["bucket", "fastrand"])
def test_config4_copurchase_like_every_width(es, mode):
    from gpu_util import check_every_element
    w, d = _cfg4_device()
    for W in w.Ws:
        worst = check_every_element(d, W, mode, 0, what=f"cfg4 {mode} W={W}")
        _say(f"cfg4 {mode} W={W}: max normalised error {worst:.2e} over all {w.N} x {w.F} elements")


def test_config4_copurchase_like_edge_lists(es):
    from gpu_util import check_edges
    w, d = _cfg4_device()
    check_edges(d, 32, "fastrand", 0)
    _say("cfg4 fastrand W=32: edge lists identical")
    check_edges(d, 128, "fastrand", 77)
    check_edges(d, 64, "bucket", 0)
    _say("cfg4 fastrand W=128 (seeded) and bucket W=64: edge lists identical")
