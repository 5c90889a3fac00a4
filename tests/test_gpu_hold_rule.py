"""GPU tier for the rule that chooses kernels whose lanes hold a row's entries:
300 MB gathered by a run, on rows of 16 lanes or more.  A matrix above the line
against its two halves below it: a row's sum does not depend on the kernel, so
the results are bitwise the same; and integer-valued inputs equal the FP64
oracle bit for bit above it."""
import numpy as np
import pytest

from gpu_util import device_B, exact
from paper_2606_22482_amd import api, synth
from test_gpu_held_entries import EDGES, rows_of

pytestmark = pytest.mark.gpu

LINE = 300e6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,kind", [(64, "f32"), (130, "f32"), (200, "f32"), (128, "f16"), (130, "bf16"), (260, "bf16"),
                                    (520, "f16")])
def test_above_equals_below(n, kind):
    import torch
    rng = np.random.default_rng(n)
    size = 4 if kind == "f32" else 2
    want = int(LINE / (n * size)) + 1
    half = list(rng.permutation(EDGES * (want // (2 * sum(EDGES)) + 1)))
    A = rows_of(half * 2, 900, kind, 3 + n)
    cut = len(half)
    assert A.colidx.size * n * size >= LINE > int(A.rowptr[cut]) * n * size
    lo = synth.CSR(cut, A.k, A.rowptr[:cut + 1], A.colidx[:A.rowptr[cut]], A.vals[:A.rowptr[cut]], kind)
    e = int(A.rowptr[cut])
    hi = synth.CSR(A.m - cut, A.k, A.rowptr[cut:] - e, A.colidx[e:], A.vals[e:], kind)
    Bf = device_B(synth.dense_values(rng, (A.k, n), kind), kind)
    B = synth.int_dense(9 + n, (A.k, n), -8, 8, kind=kind)
    for pipe in (1, 2, 3):
        for ex in (1, 2):
            print("case", kind, n, pipe, ex, flush=True)
            o = api.default_opts(mode="plain", pipeline=pipe, exec=ex, seg_len=64)
            got = []
            for M in (A, lo, hi):
                p = api.Plan(M, n, kind, o)
                C = torch.full((M.m, n), float("nan"), device="cuda")
                p.run(Bf, C)
                if M is A:
                    Ci = torch.full((M.m, n), float("nan"), device="cuda")
                    p.run(device_B(B, kind), Ci)
                torch.cuda.synchronize()
                got.append(C)
            exact(Ci, A, B, kind)
            assert torch.equal(got[0], torch.cat(got[1:]))
