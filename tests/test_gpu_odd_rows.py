"""GPU tier for rows that are not whole chunks under options that change how they
are read: cache policies of cold rows, and panels of a number of columns that is
no multiple of a chunk, alone and without allocation.  Integer-valued inputs
equal the FP64 oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import device_B, exact
from paper_2606_22482_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("policy", [2, 16, 18])
@pytest.mark.parametrize("n,kind", [(9, "bf16"), (47, "f16"), (131, "bf16"), (48, "f16"), (47, "f32"), (5, "bf16")])
def test_cold_policies(n, kind, policy):
    import torch
    A = synth.random_csr(900, 700, 0.05, n + policy, val_kind=kind, int_values=(-2, 2), empty_rows=0.1)
    B = synth.int_dense(n, (A.k, n), -8, 8, kind=kind)
    for mode in ("plain", "mixed"):
        for hot in (0, 100):
            for pad in (0, 1):
                print("case", n, kind, policy, mode, hot, pad, flush=True)
                p = api.Plan(A, n, kind, api.default_opts(mode=mode, cold_policy=policy, hot_cols=hot, seg_len=30))
                assert p.stats()["opts"]["cold_policy"] == policy
                C = torch.full((A.m, n), float("nan"), device="cuda")
                p.run(device_B(B, kind, pad_cols=pad), C)
                torch.cuda.synchronize()
                exact(C, A, B, kind)
