"""GPU tier for windows that gather more rows of B for their remainders than for
their tiles: a lane group takes one row or four, by the number of waves.  Rows
of 0 to 90 remainder entries (the edges of what a step and a load of entries
hold), widths around the panels and odd ones.  Integer-valued inputs equal the
FP64 oracle bit for bit; every launch form and a batch give the same bits of
float inputs."""
import numpy as np
import pytest

from gpu_util import device_B, exact
from paper_2606_22482_amd import api, synth

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 47, 90]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def blocks_and_strays(m, k, kind, seed):
    """Every 16 rows share 24 columns below 24 * blocks; each row has further
    single columns above them, as many as EDGES says in turn."""
    rng = np.random.default_rng(seed)
    cols, ptr = [], [0]
    base = k // 2
    for r in range(m):
        n = EDGES[int(rng.integers(len(EDGES)))]
        own = (r // 16 * 24 % (base - 24)) + np.flatnonzero(rng.random(24) < 0.8)
        cols.append(np.concatenate([own, base + np.sort(rng.choice(k - base, n, replace=False))]))
        ptr.append(ptr[-1] + len(cols[-1]))
    vals = rng.integers(-2, 3, size=ptr[-1]).astype(np.float32)
    if kind == "bf16":
        vals = synth.to_bf16_bits(vals)
    elif kind == "f16":
        vals = vals.astype(np.float16).view(np.uint16)
    return synth.CSR(m, k, np.array(ptr, np.int64), np.concatenate(cols).astype(np.int32), vals, kind)


# (rows, window height, widths): few waves, and more than the rule's 5000 (16-bit) or 700 (f32)
CASES = [(500, 16, (2, 17, 32, 33, 64, 100, 128, 200, 258)), (1100, 64, (16, 64, 130)), (81000, 16, (32, 65, 128))]


@pytest.mark.parametrize("kind", [("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16"), ("f16", "f16")])
@pytest.mark.parametrize("m,h,widths", CASES)
def test_remainders(kind, m, h, widths):
    import torch
    A = blocks_and_strays(m, 4000, kind[0], m + h)
    for n in widths:
        B = synth.int_dense(n, (A.k, n), -8, 8, kind=kind[1])
        Bi, Bf = device_B(B, kind[1]), device_B(synth.dense_values(np.random.default_rng(n), (A.k, n), kind[1]), kind[1])
        outs = []
        for ex in (1, 2, 3):
            for seg in (40, 256):
                print("case", kind, m, h, n, ex, seg, flush=True)
                p = api.Plan(A, n, kind[1], api.default_opts(mode="mixed", row_order="original_ranges", window_h=h, t_row=-1,
                                                             alpha=0.2, exec=ex, seg_len=seg))
                s = p.stats()
                assert s["windows"] in (m // h, m // h + 1) and s["work_winrem"] > 3 * 32 * s["tiles"]
                C = torch.full((m, n), float("nan"), device="cuda")
                p.run(Bi, C)
                torch.cuda.synchronize()
                exact(C, A, B, kind[1])
                C = torch.full((m, n), float("nan"), device="cuda")
                p.run(Bf, C)
                Cb = torch.full((m, n), float("nan"), device="cuda")
                api.spmm_wait(api.spmm_submit([api.WorkItem(p, Bf, Cb)]))
                torch.cuda.synchronize()
                assert torch.equal(C, Cb)
                outs.append((seg, C))
        for seg, C in outs:
            assert torch.equal(C, next(c for q, c in outs if q == seg))
