"""GPU tier for the windows of a batch: its panels and waves are chosen for all of
its plans together, so a plan's windows run in other shapes than alone (64-row
windows in panels of 128 by two blocks a wave, narrower panels and other splits
alone), with the same bits; integer-valued inputs equal the FP64 oracle."""
import numpy as np
import pytest

from gpu_util import device_B, exact
from paper_2606_22482_amd import api, synth
from test_gpu_window_remainders import blocks_and_strays

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("h,alpha", [(64, 0.0), (64, 0.05), (32, 0.05), (16, 0.2)])
@pytest.mark.parametrize("kind,widths", [(("bf16", "bf16"), (128, 200, 131)), (("f16", "f16"), (64, 256)),
                                         (("f32", "bf16"), (100,)), (("f32", "f32"), (64, 100))])
def test_batch_equals_alone(kind, widths, h, alpha):
    """Six plans of 120 windows (alpha 0: every entry in tiles; else long
    remainders), together more than the 700 items that keep the widest panels."""
    import torch
    items, alone = [], []
    for i in range(6):
        n = widths[i % len(widths)]
        A = blocks_and_strays(120 * h, 3000, kind[0], 11 * i + h)
        p = api.Plan(A, n, kind[1], api.default_opts(mode="mixed", row_order="original_ranges", window_h=h, t_row=-1,
                                                     alpha_c=0.0 if alpha == 0 else -1.0, alpha=alpha, seg_len=60))
        assert p.stats()["windows"] == 120
        B = synth.int_dense(n + i, (A.k, n), -8, 8, kind=kind[1])
        for x in (device_B(B, kind[1]), device_B(synth.dense_values(np.random.default_rng(i), (A.k, n), kind[1]), kind[1])):
            C = torch.full((A.m, n), float("nan"), device="cuda")
            print("case", kind, n, h, alpha, i, flush=True)
            p.run(x, C)
            torch.cuda.synchronize()
            items.append(api.WorkItem(p, x, torch.full((A.m, n), float("nan"), device="cuda")))
            alone.append((C, A, B))
    api.spmm_wait(api.spmm_submit(items))
    torch.cuda.synchronize()
    for j, (it, (C, A, B)) in enumerate(zip(items, alone)):
        assert torch.equal(it.C, C), j
        if j % 2 == 0:
            exact(it.C, A, B, kind[1])
