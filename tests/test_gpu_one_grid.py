"""GPU tier for exec 3: a plan with windows and vector rows whose rows hold a
16-byte chunk runs in one grid at any size (f32 B of any width, 16-bit B of more
than 64 columns), odd 16-bit widths included; the timer names the kernel.
Integer-valued inputs equal the FP64 oracle bit for bit, float inputs give the
bits of the serial kernels."""
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


@pytest.mark.parametrize("h,alpha", [(16, 0.2), (64, 0.05)])
@pytest.mark.parametrize("kind,n", [(("f32", "f32"), 4), (("f32", "f32"), 16), (("f32", "f32"), 63), (("f32", "f32"), 200),
                                    (("f32", "bf16"), 65), (("bf16", "bf16"), 100), (("f16", "f16"), 128),
                                    (("f16", "f16"), 257)])
def test_runs_in_one_grid(kind, n, h, alpha):
    import torch
    # rows of 24 columns and more in windows, the others vector rows
    A = blocks_and_strays(2000, 4000, kind[0], 7 + n)
    B = synth.int_dense(n, (A.k, n), -8, 8, kind=kind[1])
    Bi, Bf = device_B(B, kind[1]), device_B(synth.dense_values(np.random.default_rng(n), (A.k, n), kind[1]), kind[1])
    for pipe in (2, 3):
        for t_row in (24, 40):  # most and few of the rows in windows
            o = dict(mode="mixed", row_order="original_ranges", window_h=h, t_row=t_row, alpha=alpha, pipeline=pipe, seg_len=50)
            print("case", kind, n, h, pipe, t_row, flush=True)
            p = api.Plan(A, n, kind[1], api.default_opts(exec=3, **o))
            s = p.stats()
            assert s["windows"] > 0 and s["vector_items"] > 0
            C = torch.full((A.m, n), float("nan"), device="cuda")
            timer = api.Timer(8)
            p.run_timed(Bi, C, timer)
            torch.cuda.synchronize()
            exact(C, A, B, kind[1])
            assert [k for k, _ in timer.read()] == ["one_grid"]
            p.run(Bf, C)
            Cs = torch.full((A.m, n), float("nan"), device="cuda")
            api.Plan(A, n, kind[1], api.default_opts(exec=1, **o)).run(Bf, Cs)
            torch.cuda.synchronize()
            assert torch.equal(C, Cs)
