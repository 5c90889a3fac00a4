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


@pytest.mark.parametrize("n,panel,kind", [(47, 7, "f32"), (47, 46, "f32"), (33, 1, "f32"), (47, 15, "f16"), (131, 60, "bf16"),
                                          (48, 10, "f32"), (6, 5, "f32")])
def test_panels(n, panel, kind):
    """12,500 rows of two segments each: 7 panels of them have 175,000 arrival
    counters, which the run without allocation holds; 12 would have 300,000."""
    import torch
    rng = np.random.default_rng(n)
    m, k = 12500, 600
    col = np.sort(rng.integers(0, k, size=(m, 8)), axis=1).astype(np.int32).ravel()
    val = rng.integers(-2, 3, size=m * 8).astype(np.float32)
    val = synth.to_bf16_bits(val) if kind == "bf16" else val.astype(np.float16).view(np.uint16) if kind == "f16" else val
    A = synth.CSR(m, k, np.arange(0, 8 * m + 1, 8, dtype=np.int64), col, val, kind)
    B = synth.int_dense(n, (k, n), -8, 8, kind=kind)
    Bd = device_B(B, kind)
    p = api.Plan(A, n, kind, api.default_opts(mode="plain", n_panel=panel, seg_len=4))
    assert p.stats()["segments"] == 2 * m
    print("case", n, panel, kind, flush=True)
    for noalloc in (False, True):
        if noalloc and -(-n // panel) * 2 * m * 4 > 1 << 20:
            continue  # (more counters than it holds at one column a lane as well)
        C = torch.full((m, n), float("nan"), device="cuda")
        (p.run_noalloc if noalloc else p.run)(Bd, C)
        torch.cuda.synchronize()
        exact(C, A, B, kind)
