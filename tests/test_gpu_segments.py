"""The segmented build of large k-D tables against the binned one, which a
small record budget selects: at the rows from which on it is taken, in several
batches, for two, three and four joins."""
import os

import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu

M = 1 << 20


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _keys(torch, rng, n, k, kind):
    if kind == "wide":
        return [torch.from_numpy(rng.integers(-2**62, 2**62, n) if m % 2 else
                                 rng.integers(0, 2**33, n)).cuda() for m in range(k)]
    if kind == "one":
        return [torch.full((n,), 12345, dtype=torch.int64, device="cuda")] * k
    return [torch.from_numpy(W.fk_column(rng, n, 300_000, 1.05, rng.permutation(300_000))
                             .astype(np.int32)).cuda() for _ in range(k)]


def _build(C, torch, n, cols, preds, keys, seeds, d, widths, bits, budget):
    """Counters and selected rows after a build and a second one added to it,
    and the launches of the segmented build."""
    ct = torch.int32 if bits == 32 else torch.int64
    T = torch.full((d,) + tuple(widths), 7, dtype=ct, device="cuda")
    ns = torch.full((1,), 3, dtype=torch.int64, device="cuda")
    assert "COMPASS_2D_RECORD_BYTES" not in os.environ
    if budget:
        os.environ["COMPASS_2D_RECORD_BYTES"] = str(budget)
    C.profile_enable(True)
    try:
        C.sketch_build_kd(n, cols, preds, keys, seeds, T, ns, d, widths, counter_bits=bits)
        torch.cuda.synchronize()
        first = T.clone()
        C.sketch_build_kd(n, cols, preds, keys, seeds, T, ns, d, widths, counter_bits=bits,
                          accumulate=True)
        torch.cuda.synchronize()
        launches = C.profile_take("scan2d_segments")[0]
    finally:
        C.profile_enable(False)
        os.environ.pop("COMPASS_2D_RECORD_BYTES", None)
    assert torch.equal(T, 2 * first)
    return first, int(ns.item()), launches


@gpu
@pytest.mark.parametrize("widths,d,bits,n,hi,keys_are", [
    ([512, 512], 3, 32, 2 * M, None, "zipf"),        # whole chunks, one heavy tile
    ([512, 512], 3, 32, 2 * M + 1, None, "zipf"),    # a chunk and a half per block
    ([255, 16384], 2, 32, 2 * M + 4097, 64, "zipf"),  # one matrix row to a tile
    ([64, 50, 20], 3, 64, 2 * M + 1, 64, "wide"),     # widths not powers of two
    ([64, 50, 20], 3, 64, 3 * M + 4095, None, "wide"),
    ([16, 16, 16, 16], 2, 32, 8 * M + 1, None, "zipf"),
    ([13, 11, 9, 7], 3, 64, 12 * M + 5, 30, "wide"),
    ([7, 3], 5, 64, 2 * M + 9, 64, "one"),            # every row in one counter
    ([300, 100], 2, 32, 2 * M + 9, -1, "zipf"),       # no row selected
])
def test_segments(widths, d, bits, n, hi, keys_are):
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    print("[case] segments", widths, d, bits, n, hi, keys_are, flush=True)
    rng = np.random.default_rng(sum(widths) + d)
    keys = _keys(torch, rng, n, len(widths), keys_are)
    attr = torch.from_numpy(rng.integers(0, 100, n).astype(np.int32)).cuda()
    preds = [] if hi is None else [{"col": 0, "kind": "range", "lo": 5 if hi > 0 else 200,
                                    "hi": hi if hi > 0 else 300}]
    seeds = list(W.draw_seeds(rng, len(widths), d))
    args = (C, torch, n, [attr] if preds else [], preds, keys, seeds, d, widths, bits)
    got, ns, launches = _build(*args, None)
    ref, nr, none = _build(*args, 4 * d * M)
    assert (launches, none) == (2, 0)
    assert ns == nr
    assert torch.equal(got, ref)


@gpu
@pytest.mark.parametrize("hi", [None, 49, 1])
@pytest.mark.parametrize("bits", [32, 64])
def test_segments_in_batches(hi, bits):
    """Two full batches and a short ragged one with its own blocks and
    chunks; later batches add to the first."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    d, widths = 3, [200, 150]
    n = 2 * 2 * M + 100_003
    print("[case] segments in batches", hi, bits, n, flush=True)
    rng = np.random.default_rng(bits + (hi or 0))
    keys = _keys(torch, rng, n, 2, "zipf")
    attr = torch.from_numpy(rng.integers(0, 100, n).astype(np.int32)).cuda()
    preds = [] if hi is None else [{"col": 0, "kind": "range", "lo": 0, "hi": hi}]
    seeds = list(W.draw_seeds(rng, 2, d))
    args = (C, torch, n, [attr] if preds else [], preds, keys, seeds, d, widths, bits)
    got, ns, launches = _build(*args, 4 * d * 2 * M)
    whole, nw, one = _build(*args, None)
    ref, nr, none = _build(*args, 4 * d * M)
    assert (launches, one, none) == (6, 2, 0)
    assert ns == nw == nr
    assert torch.equal(got, ref) and torch.equal(whole, ref)


@gpu
@pytest.mark.parametrize("widths,n,dtype,segments", [
    ([64, 64], 2 * M - 1, 32, 0), ([64, 64], 2 * M, 64, 1),
    ([8, 8, 8, 8], 8 * M - 1, 32, 0), ([8, 8, 8, 8], 8 * M, 32, 1),
    ([8, 8, 8, 8], 8 * M, 64, 0), ([8, 8, 8, 8], 12 * M, 64, 1),
])
def test_rows_from_which_on(widths, n, dtype, segments):
    """Which build takes a batch, by its rows, joins and key types."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    print("[case] segments from", widths, n, dtype, flush=True)
    dt = torch.int32 if dtype == 32 else torch.int64
    keys = [torch.arange(n, device="cuda").remainder_(1000 + k).to(dt)
            for k in range(len(widths))]
    seeds = list(W.draw_seeds(np.random.default_rng(1), len(widths), 1))
    _, ns, launches = _build(C, torch, n, [], [], keys, seeds, 1, widths, 64, None)
    assert ns == 2 * n and launches == 2 * segments
