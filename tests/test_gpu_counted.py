"""Counted builds (tables without predicates whose key columns hold few
distinct keys): bit-exact against the oracle, and against the same build
through the fixed-scratch entry point, which hashes every row."""
import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu

N = 3_600_007          # times 14 sketch rows: above the counted build's floor
TILE, BIN = 16384, 16384


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _zipf(rng, n, domain, s=1.0):
    return W.fk_column(rng, n, domain, s, rng.permutation(domain), np.int64)


def _column(name, rng, n):
    """A key column by name; every one takes int64 values."""
    if name == "zipf":
        return _zipf(rng, n, 300_000)
    if name == "bin_edges":      # first and last key of each of 20 bins
        edge = np.concatenate([np.arange(20) * BIN, np.arange(20) * BIN + BIN - 1])
        return rng.choice(edge, size=n)
    if name == "one_key":
        return np.full(n, 777, dtype=np.int64)
    if name == "two_heavy":      # two heavy keys of one bin among spread ones
        k = rng.integers(0, 200_000, size=n)
        u = rng.random(n)
        k[u < 0.3] = 5
        k[u > 0.8] = 9
        return k
    if name == "sorted":
        return np.sort(_zipf(rng, n, 50_000))
    if name == "runs":           # runs of 1 to 9 equal keys
        k = np.repeat(rng.integers(0, 400_000, size=n), rng.integers(1, 10, size=n))
        return k[:n]
    if name == "few_outside":    # listed one by one: negative, 2^31 and more
        k = _zipf(rng, n, 100_000)
        k[::1000] = -3
        k[5::1500] = (1 << 31) - 1
        return k
    if name == "wide":           # low words in range, high words not
        k = _zipf(rng, n, 100_000)
        k[7::900] += 1 << 32
        k[8::900] = -(1 << 63)
        k[9::900] = (1 << 61) - 1
        return k
    if name == "late_outside":   # none in the sample, more than the list holds
        k = _zipf(rng, n, 1000)
        step = n // 1024
        at = np.arange(n)
        k[(at % step > step // 4) & (at % step < step // 3)] = 2_000_000_000
        return k
    assert name == "unique"
    return rng.permutation(n)


def _build(C, torch, n, keys, seeds, d, w, bits, accumulate=False, noalloc=False):
    cdt = torch.int32 if bits == 32 else torch.int64
    cnt = [torch.full((d, w), 11, dtype=cdt, device="cuda") for _ in keys]
    ns = torch.full((1,), 5, dtype=torch.int64, device="cuda")
    C.sketch_build(n, [], [], keys, seeds, cnt, ns, d, w, bits,
                   accumulate=accumulate, noalloc=noalloc)
    torch.cuda.synchronize()
    return [c.cpu().numpy().astype(np.int64) for c in cnt], int(ns.item())


@gpu
@pytest.mark.parametrize("name,dtype", [
    ("zipf", 32), ("zipf", 64), ("bin_edges", 32), ("one_key", 64),
    ("two_heavy", 32), ("sorted", 32), ("runs", 64), ("few_outside", 32),
    ("wide", 64), ("late_outside", 32), ("unique", 32)])
def test_counted_column(oracle, name, dtype):
    """One column hashed into two sketches, against the oracle."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(sum(map(ord, name)) + dtype)
    d, w = 7, (4096 if dtype == 32 else 3001)
    col = _column(name, rng, N).astype(np.int32 if dtype == 32 else np.int64)
    print("[case] counted", name, dtype, "n", N, "d", d, "w", w, flush=True)
    seeds = [W.draw_seeds(rng, 1, d)[0] for _ in range(2)]
    key = torch.from_numpy(col).cuda()
    got, ns = _build(C, torch, N, [key, key], seeds, d, w, 32)
    assert ns == N
    tb = W.Table("t", {"k": col})
    n_o, ref = oracle.build_table_sketches(tb, ["k", "k"], seeds, d, w)
    assert n_o == N
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)


@gpu
@pytest.mark.parametrize("order,bits,accumulate", [
    ("zipf,unique,zipf", 64, False), ("late_outside,zipf,late_outside", 32, True),
    ("sorted,few_outside,two_heavy", 32, False), ("wide,wide,wide,wide", 64, True)])
def test_counted_mixed_columns(order, bits, accumulate):
    """Counted, partly counted and uncounted columns of one table, sketches
    of a column not adjacent, a ragged last tile: equal to hashing every
    row."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    names = order.split(",")
    rng = np.random.default_rng(len(order))
    n = 8 * TILE * 55 + 1
    d, w = 11, 2048
    cols = {}
    for k in names:
        if k not in cols:
            c = _column(k, rng, n)
            cols[k] = torch.from_numpy(c if bits == 64 else c.astype(np.int32)).cuda()
    keys = [cols[k] for k in names]
    seeds = [W.draw_seeds(rng, 1, d)[0] for _ in names]
    print("[case] counted mixed", order, "n", n, "d", d, "w", w, bits, flush=True)
    got, ns = _build(C, torch, n, keys, seeds, d, w, bits, accumulate)
    ref, nr = _build(C, torch, n, keys, seeds, d, w, bits, accumulate, noalloc=True)
    assert ns == nr == (n + 5 if accumulate else n)
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)


@gpu
@pytest.mark.parametrize("order", ["zipf,zipf,sorted", "runs,few_outside,runs"])
def test_counted_second_column(order):
    """A column below the floor is counted along with one above it: equal to
    hashing every row."""
    torch = _torch()
    from paper_2102_02440_amd import compass as C
    names = order.split(",")
    rng = np.random.default_rng(len(order))
    d, w = 7, 4096
    cols = {k: torch.from_numpy(_column(k, rng, N).astype(np.int32)).cuda()
            for k in dict.fromkeys(names)}
    keys = [cols[k] for k in names]
    seeds = [W.draw_seeds(rng, 1, d)[0] for _ in names]
    print("[case] counted second", order, "n", N, "d", d, "w", w, flush=True)
    got, ns = _build(C, torch, N, keys, seeds, d, w, 32)
    ref, nr = _build(C, torch, N, keys, seeds, d, w, 32, noalloc=True)
    assert ns == nr == N
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)
