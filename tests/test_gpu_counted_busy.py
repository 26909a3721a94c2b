"""Counted builds whose column is found unfit only while its rows are being
partitioned, on a GPU that another stream keeps busy, so that workgroups of
the partition start after the flag is raised: equal to hashing every row."""
import numpy as np
import pytest

from paper_2102_02440_amd import workloads as W

gpu = pytest.mark.gpu


@gpu
@pytest.mark.parametrize("dtype", [32, 64])
def test_flag_raised_while_workgroups_wait(dtype):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(dtype)
    n, d, w = 16_000_001, 7, 4096
    print("[case] flag raised meanwhile", dtype, "n", n, "d", d, "w", w, flush=True)
    # none of the 1024 sampled rows outside, a thirtieth of the others: the
    # list of outside keys (n / 32 of them) overflows near the end
    k = rng.integers(0, 100_000, n)
    step = n // 1024
    at = np.arange(n) % step
    k[(at > step // 4) & (at < step // 4 + step // 28)] = 2_000_000_000
    dt = torch.int32 if dtype == 32 else torch.int64
    key = torch.from_numpy(k).to(dt).cuda()
    attr = torch.from_numpy(rng.integers(0, 100, n).astype(np.int32)).cuda()
    seeds = [W.draw_seeds(rng, 1, d)[0] for _ in range(2)]

    def build(preds, noalloc=False):
        cnt = [torch.zeros((d, w), dtype=torch.int32, device="cuda") for _ in seeds]
        ns = torch.zeros(1, dtype=torch.int64, device="cuda")
        C.sketch_build(n, [attr] if preds else [], preds, [key, key], seeds, cnt, ns, d, w,
                       32, noalloc=noalloc)
        return cnt, ns

    ref, nr = build([], noalloc=True)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    got = []
    for _ in range(4):
        with torch.cuda.stream(side):
            build([{"col": 0, "kind": "range", "lo": 0, "hi": 89}])
        got.append(build([]))
    torch.cuda.synchronize()
    for cnt, ns in got:
        assert ns.item() == nr.item() == n
        for a, b in zip(cnt, ref):
            assert torch.equal(a, b)
