"""GPU tier for window items: the number of waves a window is split over, the
panel widths, odd tile counts and remainders longer than what an item holds in
flight (16 entries a row).  Integer-valued inputs (every sum exact in FP32), so
the result equals the FP64 oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import exact
from paper_2606_22482_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# rows, k, density, alpha: one, two and four waves a 64-row window (enough long
# windows, enough short ones, few); tiles beside long remainders, mostly at 16
# rows and at 64
SHAPES = [
    (45000, 2600, 0.012, 0.0),
    (45000, 150, 0.05, 0.0),
    (1000, 700, 0.05, 0.0),
    (1500, 900, 0.06, 0.11),
    (1500, 900, 0.06, 0.06),
]


# (the large shapes at the widths that reach a new split)
CASES = [(s, n) for s in range(len(SHAPES)) for n in ((64, 128) if s < 2 else (1, 17, 32, 64, 100, 128, 200))]


@pytest.mark.parametrize("shape,n", CASES)
@pytest.mark.parametrize("kind", [("f32", "f32"), ("bf16", "bf16"), ("f32", "bf16")])
def test_window_shapes(kind, shape, n):
    import torch
    m, k, density, alpha = SHAPES[shape]
    A = synth.random_csr(m, k, density, 7 + n, val_kind=kind[0], int_values=(-2, 2), empty_rows=0.05)
    B = synth.int_dense(9 + n, (A.k, n), -8, 8, kind=kind[1])
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind[1]]
    Bd = (torch.from_numpy(B) if kind[1] == "f32" else torch.from_numpy(B.view(np.int16)).view(dt)).cuda()
    for h in (16, 32, 64):
        for ex in (1, 2, 3):
            print("case", kind, SHAPES[shape], n, h, ex, flush=True)
            p = api.Plan(A, n, kind[1], api.default_opts(mode="mixed", window_h=h, t_row=-1, alpha_c=0.0, alpha=alpha,
                                                         exec=ex))
            C = torch.full((A.m, n), float("nan"), device="cuda")
            p.run(Bd, C)
            torch.cuda.synchronize()
            exact(C, A, B, kind[1])
