"""Calls that take more scratch than their plain way (counted builds, AGMS
sign tables, the node groups of an estimate) where the pool cannot grow: the
device has no room for more (COMPASS_SCRATCH_BYTES stands in for that), or the
stream is being captured.  Results are those of the unlimited call."""
import contextlib
import os

import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@contextlib.contextmanager
def _limit(C, n_bytes):
    """An empty pool that grows to n_bytes at most."""
    C.release()
    os.environ["COMPASS_SCRATCH_BYTES"] = str(n_bytes)
    try:
        yield
    finally:
        del os.environ["COMPASS_SCRATCH_BYTES"]
        C.release()


def _counted_args(torch, rng, n=4_000_003, d=7, w=4096):
    key = torch.from_numpy(W.fk_column(rng, n, 200_000, 1.0, rng.permutation(200_000))).cuda()
    return n, key, [W.draw_seeds(rng, 1, d)[0] for _ in range(2)], d, w


def _counted(C, torch, args, noalloc=False, out=None):
    n, key, seeds, d, w = args
    cnt, ns = out or ([torch.full((d, w), 5, dtype=torch.int32, device="cuda") for _ in seeds],
                      torch.full((1,), 9, dtype=torch.int64, device="cuda"))
    C.sketch_build(n, [], [], [key, key], seeds, cnt, ns, d, w, 32, noalloc=noalloc)
    return cnt, ns


@gpu
def test_counted_build_without_room(oracle):
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    args = _counted_args(torch, np.random.default_rng(3))
    ref, nr = _counted(C, torch, args, noalloc=True)
    torch.cuda.synchronize()
    # the counted build's slab alone: 256 chunks of 14 x 4096 int32; the fused
    # scan's takes a quarter of it
    for limit, counts in ((256 * 14 * 4096 * 4, False), (4 << 30, True)):
        print("[case] counted, scratch", limit, flush=True)
        with _limit(C, limit):
            C.profile_enable(True)
            try:
                for _ in range(2):
                    got, ns = _counted(C, torch, args)
                torch.cuda.synchronize()
                launches = C.profile_take("count")[0]
            finally:
                C.profile_enable(False)
        assert launches == (2 if counts else 0)
        assert ns.item() == nr.item() == args[0]
        for a, b in zip(got, ref):
            assert torch.equal(a, b)


@gpu
def test_pool_grows_to_what_is_needed():
    """A pool that cannot double still grows to the size of the call."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(4)
    n, d = 3_000_000, 3
    keys = torch.from_numpy(rng.integers(0, n, n).astype(np.int32)).cuda()
    seeds = [W.draw_seeds(rng, 1, d)[0]]
    out = []
    print("[case] pool that cannot double", flush=True)
    for limited in (False, True):
        with (_limit(C, 160 << 20) if limited else contextlib.nullcontext()):
            for w in (4096, 8192, 16384):   # slabs of 25, 50 and 100 MB at most
                cnt = [torch.zeros((d, w), dtype=torch.int32, device="cuda")]
                ns = torch.zeros(1, dtype=torch.int64, device="cuda")
                C.sketch_build(n, [], [], [keys], seeds, cnt, ns, d, w, 32)
                torch.cuda.synchronize()
                out.append(cnt[0].cpu())
    for a, b in zip(out[:3], out[3:]):
        assert torch.equal(a, b)


@gpu
def test_small_table_without_room(oracle):
    """A table spread over more chunks than its tiles need, and over as few as
    fit."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(8)
    n, d, w = 130_001, 3, 16384
    col = rng.integers(0, n, n).astype(np.int32)
    key = torch.from_numpy(col).cuda()
    seeds = [W.draw_seeds(rng, 1, d)[0]]
    n_o, ref = oracle.build_table_sketches(W.Table("t", {"k": col}), ["k"], seeds, d, w)
    # slab rows of 3 x 16384 int32: the plain chunks alone, and all
    for chunks in (2, 3, 64):
        print("[case] small table, slab rows", chunks, flush=True)
        with _limit(C, chunks * d * w * 4):
            cnt = [torch.full((d, w), 3, dtype=torch.int32, device="cuda")]
            ns = torch.zeros(1, dtype=torch.int64, device="cuda")
            C.sketch_build(n, [], [], [key], seeds, cnt, ns, d, w, 32)
            torch.cuda.synchronize()
        assert ns.item() == n == n_o
        assert np.array_equal(cnt[0].cpu().numpy(), ref[0])


@gpu
def test_agms_build_without_room(oracle):
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(5)
    n, r, b = 400_000, 4, 130
    keys = [rng.integers(0, 5000, n).astype(np.int32)]
    seeds = W.draw_seeds(rng, 1, r * b)
    dk = [torch.from_numpy(k).cuda() for k in keys]
    co = oracle.agms_sketch(keys, list(seeds), r, b)
    print("[case] agms, scratch 1 MiB", flush=True)
    with _limit(C, 1 << 20):
        cnt = torch.zeros((r, b), dtype=torch.int64, device="cuda")
        ns = torch.zeros(1, dtype=torch.int64, device="cuda")
        C.agms_build(n, [], [], dk, list(seeds), cnt, ns, r, b)
        torch.cuda.synchronize()
    assert np.array_equal(cnt.cpu().numpy(), co)
    assert ns.item() == n


@gpu
@pytest.mark.parametrize("mib", [12, 3])
def test_estimate_without_room(mib):
    """All sub-plans of a seven-table tree, some of them not certified: with
    node scratch for the 26 tasks of a level (15 MiB in all), for half of them
    and for two.  Rows, estimates and flags bit for bit."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(6)
    nt, d, w = 7, 5, 1000
    eu, ev = [0, 0, 1, 1, 2, 5], [1, 2, 3, 4, 5, 6]
    sk = [torch.from_numpy(rng.integers(-99, 100, size=(d, w))).cuda() for _ in range(2 * 6)]
    n_sel = torch.full((nt,), 1 << 24, dtype=torch.int64, device="cuda")
    masks = W.connected_masks(nt, eu, ev, min_tables=2)
    print("[case] estimate, scratch", mib, "MiB, sub-plans", len(masks), flush=True)

    def run():
        row, est, flags = C.estimate(nt, eu, ev, d, w, 64, n_sel, sk, masks)
        torch.cuda.synchronize()
        return row.cpu(), est.cpu().view(torch.int64), flags.cpu()

    ref = run()
    assert len(set(ref[2].tolist())) == 2
    with _limit(C, mib << 20):
        for _ in range(2):
            for a, b in zip(run(), ref):
                assert torch.equal(a, b)


@gpu
def test_counted_build_captured_with_a_small_pool():
    """A pool warmed by a build that takes less scratch suffices to capture a
    counted one's plain way (nothing may be allocated then)."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    args = _counted_args(torch, np.random.default_rng(7))
    ref, nr = _counted(C, torch, args, noalloc=True)
    print("[case] counted build captured", flush=True)
    C.release()
    side = torch.cuda.Stream()
    n, key, seeds, d, w = args
    out = ([torch.zeros((d, w), dtype=torch.int32, device="cuda") for _ in seeds],
           torch.zeros(1, dtype=torch.int64, device="cuda"))
    with torch.cuda.stream(side):   # 8 bytes a row and sketch: above the fused slab
        C.sketch_build(n, [key], [{"col": 0, "kind": "range", "lo": 0, "hi": 9}], [key, key],
                       seeds, out[0], out[1], d, w, 32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        _counted(C, torch, args, out=out)
    for k in range(3):
        out[0][0].fill_(k)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert out[1].item() == nr.item() == args[0]
        for a, b in zip(out[0], ref):
            assert torch.equal(a, b)
    del g
    C.release()
