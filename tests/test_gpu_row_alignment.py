"""GPU tier for rows of any width and alignment: B and C rows are read and
written in 16-byte chunks at element alignment, the last chunk of a row moved
left to stay inside it.  Integer-valued inputs (every sum exact in FP32), so
the result equals the FP64 oracle bit for bit; the columns beside C's own stay
untouched."""
import numpy as np
import pytest

from gpu_util import exact
from paper_2606_22482_amd import api, synth

pytestmark = pytest.mark.gpu

KINDS = [("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16"), ("f16", "f16")]
# around one chunk (4 f32, 8 16-bit), a window panel (32, 64, 128), one and
# two chunks a lane (256 / 512) and a last panel narrower than a chunk (514)
WIDTHS = [3, 4, 5, 7, 8, 9, 31, 33, 63, 65, 127, 130, 255, 258, 514]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def offset_view(rows, cols, dtype, pad, shift, fill):
    """rows x cols inside a buffer whose row stride is cols + pad, starting
    `shift` elements into it (the buffer ends with the last row)."""
    import torch
    ld = cols + pad
    flat = torch.full((shift + max(rows - 1, 0) * ld + cols,), fill, dtype=dtype, device="cuda")
    return flat, flat.as_strided((rows, cols), (ld, 1), shift)


def run(A, B, bk, n, opts, pad_b, shift_b, pad_c, shift_c, batched=False):
    import torch
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[bk]
    src = torch.from_numpy(B) if bk == "f32" else torch.from_numpy(B.view(np.int16)).view(dt)
    _, Bd = offset_view(A.k, n, dt, pad_b, shift_b, float("nan"))
    Bd.copy_(src)
    flat, C = offset_view(A.m, n, torch.float32, pad_c, shift_c, 7.0)
    p = api.Plan(A, n, bk, api.default_opts(**opts))
    if batched:
        api.spmm_wait(api.spmm_submit([api.WorkItem(p, Bd, C)]))
    else:
        p.run(Bd, C)
    torch.cuda.synchronize()
    exact(C, A, B, bk)
    mine = torch.zeros_like(flat, dtype=torch.bool)
    mine.as_strided(C.shape, C.stride(), shift_c).fill_(True)
    assert bool((flat[~mine] == 7.0).all()), "wrote outside C"


@pytest.mark.parametrize("n", WIDTHS)
@pytest.mark.parametrize("kind", range(4))
def test_any_width_and_alignment(kind, n):
    vk, bk = KINDS[kind]
    # long rows (split), short ones and, mixed, windows with partial tiles
    A = synth.random_csr(150, 700, 0.15, 60 + n, val_kind=vk, int_values=(-2, 2), dup_frac=0.02,
                         empty_rows=0.1)
    B = synth.int_dense(80 + n, (A.k, n), -8, 8, kind=bk)
    mixed = dict(mode="mixed", window_h=16, t_row=-1, alpha_c=0.0, alpha=0.16, seg_len=40)
    for opts in (dict(mode="plain", seg_len=40), dict(mode="plain", seg_len=40, n_panel=40),
                 mixed, dict(mixed, exec=1), dict(mixed, window_h=64, alpha=0.12, n_panel=24)):
        for pads in ((0, 0, 0, 0), (1, 1, 3, 1), (2, 4, 0, 2)):
            print("case", vk, bk, n, opts, pads, flush=True)
            run(A, B, bk, n, opts, *pads)
    run(A, B, bk, n, mixed, 1, 3, 1, 1, batched=True)
