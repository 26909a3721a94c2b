"""Which AGMS builds take sign tables, by the launches' profile names, on both
sides of the line, and where the keys do not fit them; counters against the
oracle's on sampled basic sketches."""
import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu


@gpu
@pytest.mark.parametrize("n,r,b,joins,keys_are,signs", [
    (1_600_000, 1, 125, 1, "repeat", True),     # 2e8 evaluations
    (1_599_999, 1, 125, 1, "repeat", False),
    (400_000, 4, 125, 1, "repeat", True),       # four groups of sketches
    (25_000_000, 2, 5, 1, "repeat", False),     # fewer lanes than a gather costs
    (800_001, 1, 128, 2, "shared", True),       # both joins on one column
    (1_600_001, 1, 125, 1, "distinct", True),   # the device leaves the tables
])
def test_which_way(oracle, n, r, b, joins, keys_are, signs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    print("[case] agms way", n, r, b, joins, keys_are, flush=True)
    rng = np.random.default_rng(n % 1000 + b)
    if keys_are == "distinct":
        keys = [rng.integers(0, 2**40, n) for _ in range(joins)]
    else:
        keys = [rng.integers(0, 40_000, n).astype(np.int32)] * joins
    seeds = W.draw_seeds(rng, joins, r * b)
    dk = [torch.from_numpy(k).cuda() for k in keys]
    if keys_are == "shared":
        dk = [dk[0]] * joins
    cnt = torch.full((r, b), 9, dtype=torch.int64, device="cuda")
    ns = torch.full((1,), 9, dtype=torch.int64, device="cuda")
    C.profile_enable(True)
    try:
        C.agms_build(n, [], [], dk, list(seeds), cnt, ns, r, b)
        torch.cuda.synchronize()
        ways = C.profile_take("agms_signs")[0], C.profile_take("agms_direct")[0]
    finally:
        C.profile_enable(False)
    assert ways == ((1, 0) if signs else (0, 1))
    assert ns.item() == n
    got = cnt.cpu().numpy().reshape(-1)
    for c in (0, r * b // 2, r * b - 1):
        one = oracle.agms_sketch(keys, [s[c:c + 1] for s in seeds], 1, 1)
        assert got[c] == one[0, 0], c
