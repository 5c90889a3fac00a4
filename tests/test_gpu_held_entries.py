"""GPU tier for entries held by the lanes that sum a row: row lengths at the
edges of a step, of a hold (two entries a lane) and of a segment, at widths on
both sides of the rule that chooses it, alone and in a batch.  Integer-valued
inputs (every sum exact in FP32), so the result equals the FP64 oracle bit for
bit."""
import numpy as np
import pytest

from gpu_util import exact
from paper_2606_22482_amd import api, synth

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 255, 256, 257, 300, 513]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def rows_of(lengths, k, kind, seed):
    rng = np.random.default_rng(seed)
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(k, n, replace=False)) for n in lengths] or [[]]).astype(np.int32)
    val = rng.integers(-2, 3, size=col.size).astype(np.float32)
    if kind == "bf16":
        val = (val.view(np.uint32) >> 16).astype(np.uint16)
    elif kind == "f16":
        val = val.astype(np.float16).view(np.uint16)
    return synth.CSR(len(lengths), k, ptr, col, val, kind)


@pytest.mark.parametrize("n", [8, 16, 32, 33, 64, 128, 200, 256, 260, 512, 520])
@pytest.mark.parametrize("kind", [("f32", "f32"), ("bf16", "bf16"), ("f16", "f16")])
def test_row_lengths(kind, n):
    import torch
    rng = np.random.default_rng(n)
    lengths = list(rng.permutation(EDGES * 3)) + EDGES[::-1] + [3] * 70 + [600]
    A = rows_of(lengths, 900, kind[0], 3 + n)
    B = synth.int_dense(9 + n, (A.k, n), -8, 8, kind=kind[1])
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind[1]]
    Bd = (torch.from_numpy(B) if kind[1] == "f32" else torch.from_numpy(B.view(np.int16)).view(dt)).cuda()
    for pipe in (0, 2, 3):
        for ex in (1, 2):
            for seg in (64, 256, 4096):
                print("case", kind, n, pipe, ex, seg, flush=True)
                p = api.Plan(A, n, kind[1], api.default_opts(mode="plain", pipeline=pipe, exec=ex, seg_len=seg))
                C = torch.full((A.m, n), float("nan"), device="cuda")
                p.run(Bd, C)
                torch.cuda.synchronize()
                exact(C, A, B, kind[1])
                if ex == 2:
                    C.fill_(float("nan"))
                    api.spmm_wait(api.spmm_submit([api.WorkItem(p, Bd, C)]))
                    torch.cuda.synchronize()
                    exact(C, A, B, kind[1])
