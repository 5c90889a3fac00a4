"""GPU tier for rows packed by size class at widths that are not whole chunks: a
lane takes a 16-byte chunk of any row that holds one, so a row of n columns has
ceil(n / 4) (f32) or ceil(n / 8) (16-bit) chunk lanes.  Against the packed
variant, which sums rows of class 1 and of all groups in the same order: bit for
bit on those rows, within the FP32 bound of the oracle on all; f32 rows of more
than 32 such columns have these two classes only."""
import numpy as np
import pytest

from gpu_util import TOL_F32, device_B, parity
from paper_2606_22482_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("ex", [1, 2])
@pytest.mark.parametrize("n,kind", [(7, "f32"), (30, "f32"), (33, "f32"), (47, "f32"), (130, "f32"), (9, "f16"), (33, "f16"),
                                    (65, "bf16"), (100, "f16")])
def test_ragged_widths(n, kind, ex):
    import torch
    e = 4 if kind == "f32" else 8
    lanes = 1 << int(np.ceil(np.log2(-(-n // e))))
    G = 64 // lanes
    A = synth.chung_lu_graph(20000, 2.2, 20.0, 1500.0, 40 + n, val_kind=kind, values="uniform")
    B = synth.dense_values(np.random.default_rng(n), (20000, n), kind)
    Bd = device_B(B, kind)
    got = []
    for pipe in (2, 3):
        p = api.Plan(A, n, kind, api.default_opts(mode="plain", pipeline=pipe, seg_len=300, exec=ex))
        assert p.stats()["opts"]["pipeline"] == pipe
        C = torch.full((A.m, n), float("nan"), device="cuda")
        p.run(Bd, C)
        torch.cuda.synchronize()
        parity(C, A, B, kind, TOL_F32)
        got.append(C)
    length = np.diff(A.rowptr)
    if kind == "f32" and n > 32:
        same = np.ones(A.m, bool)
    else:
        same = (length <= 16) | (length > 8 * G)
        assert G <= 2 or int((~same).sum()) > 100
    same = torch.from_numpy(same).cuda()
    assert torch.equal(got[0][same], got[1][same])
