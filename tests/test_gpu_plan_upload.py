"""GPU tier for the upload of a plan's tiles: a host plan's packed values are
spread on the device.  Tiles of one entry to full, odd and even numbers of them,
every window height, values of every type (signed zeros and infinities in a
tile among them), from the builder and from a plan image; a run on another
stream straight after the upload; against the plan that the device builder
makes, bit for bit, and the FP64 oracle."""
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


def host_csr(m, k, fill, kind, seed):
    """Row r has fill(r) of the k columns, at random."""
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(k, fill(r), replace=False)) for r in range(m)]
    ptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    v = rng.integers(-3, 4, size=int(ptr[-1])).astype(np.float32)
    if kind == "bf16":
        v = synth.to_bf16_bits(v)
    elif kind == "f16":
        v = v.astype(np.float16).view(np.uint16)
    return synth.CSR(m, k, ptr, np.concatenate(cols).astype(np.int32), v, kind)


@pytest.mark.parametrize("kind", [("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16"), ("f16", "f16")])
@pytest.mark.parametrize("h", [16, 32, 64])
@pytest.mark.parametrize("m,k,fill", [(64, 32, lambda r: 32), (37, 32, lambda r: 1 + r % 3), (200, 97, lambda r: r % 98),
                                      (130, 3000, lambda r: 1 + (r * 7) % 40)])
def test_host_plan_tiles(kind, h, m, k, fill):
    import torch
    A = host_csr(m, k, fill, kind[0], m + h)
    n = 48
    B = synth.int_dense(n, (k, n), -8, 8, kind=kind[1])
    Bd = device_B(B, kind[1])
    o = api.default_opts(mode="mfma_only", row_order="original_ranges", window_h=h)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def ran(p):
        C = torch.full((m, n), float("nan"), device="cuda")
        torch.cuda.synchronize()
        p.run(Bd, C, side)
        torch.cuda.synchronize()
        return C
    print("case", kind, h, m, k, flush=True)
    host = api.Plan(A, n, kind[1], o)
    C = ran(host)
    exact(C, A, B, kind[1])
    assert torch.equal(C, ran(api.Plan.deserialize(host.serialize())))
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind[0]]
    vals = torch.from_numpy(A.vals) if kind[0] == "f32" else torch.from_numpy(A.vals.view(np.int16)).view(dt)
    dev = api.Plan.on_device(torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(A.colidx).cuda(), vals.cuda(), m, k, n,
                             kind[1], o)
    assert dev.stats()["tiles"] == host.stats()["tiles"]
    assert torch.equal(C, ran(dev))
    # the host views of both hold the same tiles
    a, b = host.export(), dev.export()
    assert np.array_equal(a["tile_bitmap"], b["tile_bitmap"]) and np.array_equal(a["tile_vals"], b["tile_vals"])


def test_special_values_reach_the_tiles():
    """-0, infinities and the largest bf16 value, alone in their rows."""
    import torch
    special = np.array([0x8000, 0x7F80, 0xFF80, 0x7F7F, 0x0080], np.uint16)
    A = synth.CSR(5, 5, np.arange(6, dtype=np.int64), np.arange(5, dtype=np.int32), special, "bf16")
    B = synth.to_bf16_bits(np.ones((5, 8), np.float32))
    p = api.Plan(A, 8, "bf16", api.default_opts(mode="mfma_only"))
    assert np.array_equal(p.export()["tile_vals"], special)
    C = torch.empty(5, 8, device="cuda")
    p.run(device_B(B, "bf16"), C)
    torch.cuda.synchronize()
    # (a column of ones: a row's own value, plus zeros from the tile's other slots)
    want = (special.astype(np.uint32) << 16).view(np.float32)
    assert np.array_equal(C.cpu().numpy(), np.repeat(want[:, None] + 0.0, 8, 1))
