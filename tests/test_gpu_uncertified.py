"""Tree sub-plans whose 128-bit row values cannot be certified: the fp64
evaluation (one twin in double per tree node, shared by the sub-plans) next
to certified sub-plans of the same call, against the oracle's exact rows."""
import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu


@gpu
@pytest.mark.parametrize("shape,d,w,bits", [
    ("chain", 5, 64, 32), ("star", 3, 33, 64), ("bushy", 7, 48, 32)])
def test_uncertified_trees(oracle, shape, d, w, bits):
    """Selected counts are declared far above the sketches' own sums (they
    only have to bound them), so the larger sub-plans are not certified while
    every |X_i| stays below 2^127.  Flags and 128-bit rows exact; the
    estimate within 1e-12 of the contraction over absolute values (2^-53
    times some hundred roundings on the longest chain of sums)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(len(shape) * 100 + d)
    nt = 6
    parent = {"chain": [0, 1, 2, 3, 4], "star": [0, 0, 0, 0, 0],
              "bushy": [0, 0, 1, 1, 2]}[shape]
    eu, ev = parent, list(range(1, nt))
    sk = [rng.integers(-40, 41, size=(d, w)).astype(np.int64) for _ in range(2 * len(eu))]
    n_sel = [1 << 30] * nt            # 2^180 for all six: four tables still certify
    dt = torch.int32 if bits == 32 else torch.int64
    dev = [torch.from_numpy(s).to(dt).cuda() for s in sk]
    masks = W.connected_masks(nt, eu, ev, min_tables=2)
    print("[case] uncertified", shape, "d", d, "w", w, bits, "sub-plans", len(masks),
          flush=True)
    row, est, flags = C.estimate(nt, eu, ev, d, w, bits,
                                 torch.tensor(n_sel, dtype=torch.int64).cuda(), dev, masks)
    torch.cuda.synchronize()
    vals, _, f_o = oracle.estimate(nt, eu, ev, d, w, sk, n_sel, masks)
    babs, _, _ = oracle.estimate(nt, eu, ev, d, w, [np.abs(s) for s in sk], n_sel, masks)
    got, est, flags = C.row_values(row), est.cpu().numpy(), flags.cpu().numpy()
    seen = set()
    for m, mask in enumerate(masks):
        exact = bin(mask).count("1") <= 4
        seen.add(exact)
        assert flags[m] == (C.FLAG_EXACT if exact else C.FLAG_APPROX) == (f_o[m] & 1 or 4)
        assert got[m] == [v & ((1 << 128) - 1) for v in vals[m]]
        med = sorted(vals[m])[d // 2]
        tol = 0.0 if exact else 1e-12 * float(max(babs[m]))
        assert abs(est[m] - float(med)) <= tol, hex(mask)
    assert seen == {True, False}
