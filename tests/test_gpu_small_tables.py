"""Tables too small to fill the GPU, without predicates: their rows and slices
spread over more workgroups, counters bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu


@gpu
@pytest.mark.parametrize("n,k,d,w,bits", [
    (1, 1, 1, 8, 32),            # one slice: nothing to spread
    (2000, 1, 7, 4096, 32),
    (8191, 3, 5, 3000, 64),      # one ragged tile
    (8193, 2, 11, 32768, 32),    # two tiles, slices that fill the LDS
    (200_001, 3, 7, 1000, 64),   # more slices than groups of one
    (70_001, 4, 13, 64, 32),     # more than one launch's slices
])
def test_small_table_without_predicates(oracle, n, k, d, w, bits):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    print("[case] small table", n, k, d, w, bits, flush=True)
    rng = np.random.default_rng(n + k + d)
    cols = {"c%d" % s: rng.integers(-5, max(2, n // 3), n).astype(np.int64 if s % 2 else np.int32)
            for s in range(k)}
    seeds = [W.draw_seeds(rng, 1, d)[0] for _ in range(k)]
    cdt = torch.int32 if bits == 32 else torch.int64
    cnt = [torch.full((d, w), 9, dtype=cdt, device="cuda") for _ in range(k)]
    ns = torch.full((1,), 4, dtype=torch.int64, device="cuda")
    keys = [torch.from_numpy(c).cuda() for c in cols.values()]
    for accumulate in (False, True):
        C.sketch_build(n, [], [], keys, seeds, cnt, ns, d, w, bits, accumulate=accumulate)
    torch.cuda.synchronize()
    n_o, ref = oracle.build_table_sketches(W.Table("t", cols), list(cols), seeds, d, w)
    assert n_o == n and int(ns.item()) == 2 * n
    for g, r in zip(cnt, ref):
        assert np.array_equal(g.cpu().numpy().astype(np.int64), 2 * r)
