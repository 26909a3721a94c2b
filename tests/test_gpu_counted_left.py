"""Counted builds that leave some columns to the row scan, whose workgroups
then share out those columns' slice groups: several launches, groups of
unequal sizes, few tiles.  Equal to hashing every row."""
import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu


@gpu
@pytest.mark.parametrize("order,n,d,w,bits", [
    ("r,u,r,u,u", 1_600_001, 11, 16384, 32),     # 30 groups: two launches
    ("u,u,u,u,r", 1_300_000, 13, 2048, 64),      # 65 slices: two launches
    ("r,r,u", 5_300_000, 7, 8192, 32),           # groups of four and three left
    ("u,r,v", 7_300_003, 7, 3000, 64),           # two columns left, apart
    ("u", 14_000_000, 5, 64, 32),                # one column, one group's LDS
    ("v,u", 1_600_000, 32, 1, 32),               # one counter a row
    ("u,r", 2_300_001, 23, 32768, 32),           # one slice a group: four launches
])
def test_columns_left_to_the_scan(order, n, d, w, bits):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    print("[case] left to the scan", order, n, d, w, bits, flush=True)
    rng = np.random.default_rng(n + d)
    cols = {"r": rng.integers(0, n // 20, n),            # fits: counted
            "u": rng.permutation(n),                     # does not
            "v": rng.integers(-2**40, 2**40, n)}
    dev = {c: torch.from_numpy(cols[c].astype(np.int64 if c == "v" else np.int32)).cuda()
           for c in set(order.split(","))}
    keys = [dev[c] for c in order.split(",")]
    seeds = [W.draw_seeds(rng, 1, d)[0] for _ in keys]
    cdt = torch.int32 if bits == 32 else torch.int64

    def build(noalloc):
        cnt = [torch.full((d, w), 3, dtype=cdt, device="cuda") for _ in keys]
        ns = torch.zeros(1, dtype=torch.int64, device="cuda")
        for accumulate in (False, True):
            C.sketch_build(n, [], [], keys, seeds, cnt, ns, d, w, bits, accumulate=accumulate,
                           noalloc=noalloc)
        torch.cuda.synchronize()
        return cnt, int(ns.item())

    C.profile_enable(True)
    try:
        got, ns = build(False)
        assert C.profile_take("count")[0] == 2
    finally:
        C.profile_enable(False)
    ref, nr = build(True)
    assert ns == nr == 2 * n
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
