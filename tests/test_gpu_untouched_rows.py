"""GPU tier for NaN and infinities in B where no entry reads: in rows that no
entry names (row 0, which masked loads may take, and the last one among them),
in the columns beside B's own, and in one column, which must reach that column
of C alone.  Every kernel's masked entries, chunks moved inside a row, padding
columns and tiles past the end: C equals, bit for bit, that of zeros in their
place."""
import numpy as np
import pytest

from paper_2606_22482_amd import api, synth
from test_gpu_window_remainders import blocks_and_strays

pytestmark = pytest.mark.gpu

BAD = [float("nan"), float("inf"), float("-inf")]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def plans():
    for pipe in (0, 1, 2, 3):
        for ex in (1, 2):
            yield dict(mode="plain", pipeline=pipe, exec=ex, seg_len=50)
    for h, alpha in ((16, 0.2), (32, 0.1), (64, 0.05), (64, 0.0)):
        for ex in (1, 2, 3):
            yield dict(mode="mixed", row_order="original_ranges", window_h=h, t_row=24, alpha=alpha, exec=ex, seg_len=50)


@pytest.mark.parametrize("kind,n", [(("f32", "f32"), 64), (("f32", "f32"), 47), (("f32", "f32"), 258), (("f32", "bf16"), 128),
                                    (("bf16", "bf16"), 33), (("bf16", "bf16"), 100), (("f16", "f16"), 7), (("f16", "f16"), 260)])
def test_nothing_leaks(kind, n):
    import torch
    A0 = blocks_and_strays(700, 1500, kind[0], n)
    # columns 1 .. 1500 of 1502: rows 0 and 1501 of B, and every 7th of the strays', are named by nothing
    col = A0.colidx + 1
    col = np.where((col > 750) & (col % 7 == 0), col - 1, col).astype(np.int32)
    A = synth.CSR(A0.m, 1502, A0.rowptr, col, A0.vals, kind[0])
    used = np.zeros(A.k, bool)
    used[col] = True
    assert not used[0] and not used[-1] and int((~used).sum()) > 50
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind[1]]
    g = torch.Generator().manual_seed(n)
    clean = torch.randn(A.k, n, generator=g).to(dt)
    free = torch.from_numpy(np.flatnonzero(~used))
    clean[free] = 0
    bad = clean.clone()
    for i, r in enumerate(free.tolist()):
        bad[r] = BAD[i % 3]
    one = bad.clone()
    one[:, n // 2] = float("nan")

    def wide(x, fill, pad):
        t = torch.full((A.k, n + pad), fill, dtype=dt)
        t[:, :n] = x
        return t.cuda()[:, :n]
    other = torch.arange(n) != n // 2
    hit = torch.from_numpy(np.diff(A.rowptr) > 0)
    for o in plans():
        print("case", kind, n, o, flush=True)
        p = api.Plan(A, n, kind[1], api.default_opts(**o))

        def ran(x, batch=False):
            C = torch.full((A.m, n), 5.0, device="cuda")
            if batch:
                api.spmm_wait(api.spmm_submit([api.WorkItem(p, x, C)]))
            else:
                p.run(x, C)
            torch.cuda.synchronize()
            return C.cpu()
        want = ran(wide(clean, 0.0, 0))
        assert bool(torch.isfinite(want).all())
        for pad in (0, 2, 3):
            assert torch.equal(want, ran(wide(bad, float("nan"), pad)))
        assert torch.equal(want, ran(wide(bad, float("nan"), 2), batch=True))
        C = ran(wide(one, float("inf"), 1))
        assert torch.equal(want[:, other], C[:, other]) and bool(torch.isnan(C[hit, n // 2]).all())
