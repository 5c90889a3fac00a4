"""GPU tier for 64-row windows whose wave takes several 16-row blocks: all four
(enough long windows) or two (enough short ones), in panels of 128, 64 and 32
columns, through a buffer resource and by plain loads (odd 16-bit widths), with
remainders of 0 to 40 entries a row, split rows, and partial items.  (The shapes
of test_gpu_window_shapes give two and four waves a window and, where they give
two, no remainders.)  The split follows from the plan's counts, checked here.
Integer-valued inputs equal the FP64 oracle bit for bit."""
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


def shared_and_stray(windows, shared, per_row, strays, kind, seed):
    """Rows of `per_row` of `shared` columns (drawn again for each row: a column
    is seldom alone in its window) and up to `strays` single ones above them."""
    rng = np.random.default_rng(seed)
    m, k = 64 * windows, shared + 3000
    rows = np.arange(m, dtype=np.int64)
    cnt = rng.integers(0, strays + 1, size=m)
    key = np.concatenate([(rows[:, None] * k + rng.integers(0, shared, size=(m, per_row))).ravel(),
                          np.repeat(rows, cnt) * k + shared + rng.integers(0, 3000, size=int(cnt.sum()))])
    key = np.unique(key)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(key // k, minlength=m))]).astype(np.int64)
    v = rng.integers(-2, 3, size=key.size).astype(np.float32)
    v = synth.to_bf16_bits(v) if kind == "bf16" else v.astype(np.float16).view(np.uint16) if kind == "f16" else v
    return synth.CSR(m, k, ptr, (key % k).astype(np.int32), v, kind)


# blocks a wave: (windows, shared columns, of them a row, strays, partial items)
SHAPES = {
    4: [(705, 2100, 90, 14, False), (705, 2900, 120, 40, True)],
    2: [(705, 500, 24, 7, False), (705, 900, 40, 10, True)],
}


@pytest.mark.parametrize("blocks,shape", [(b, i) for b, s in SHAPES.items() for i in range(len(s))])
@pytest.mark.parametrize("kind,widths", [(("bf16", "bf16"), (128, 131, 32)), (("f16", "f16"), (64, 100)),
                                         (("f32", "bf16"), (128, 33)), (("f32", "f32"), (64, 20))])
def test_blocks_a_wave(kind, widths, blocks, shape):
    import torch
    windows, shared, per_row, strays, parts = SHAPES[blocks][shape]
    A = shared_and_stray(windows, shared, per_row, strays, kind[0], 3 + shape)
    for n in widths:
        B = synth.int_dense(n, (A.k, n), -4, 4, kind=kind[1])
        Bd = device_B(B, kind[1])
        for ex, seg in ((1, 256), (1, 12), (2, 12)):
            print("case", kind, n, blocks, shape, ex, seg, flush=True)
            p = api.Plan(A, n, kind[1], api.default_opts(mode="mixed", row_order="original_ranges", window_h=64, t_row=-1,
                                                         alpha_c=1 / 64, alpha=0.0, exec=ex, seg_len=seg))
            s, d = p.stats(), p.export()
            items, panels = s["windows"] + d["wpart_win"].size, -(-n // 128)
            assert s["windows"] == windows
            if n <= 128:  # (over two panels an item takes twice the tiles)
                assert (d["wpart_win"].size > 0) == parts
            assert 0 < s["nnz_remainder"] <= 32 * s["tiles"]
            assert items * panels >= (1100 if d["wpart_win"].size else 700)
            assert (s["tiles"] >= 32 * items) == (blocks == 4)
            C = torch.full((A.m, n), float("nan"), device="cuda")
            p.run(Bd, C)
            torch.cuda.synchronize()
            exact(C, A, B, kind[1])
