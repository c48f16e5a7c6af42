"""GPU parity of fw_dense_topk's general path (any dtype and shape) at the
edges of its tiles: row tiles of 16, key blocks of 32 and 16, column slices of
64 and 128, key splits, the selection's register and list limits, rows that
fall back to the radix selection, unaligned operands, masked keys and values
that are not finite."""
import numpy as np
import pytest

from paper_2608_25230_amd import workloads as W
from tests.parity import t2np
from tests.test_gpu_dense_topk import _compare, _oracle_rows, torch_fw  # noqa: F401

pytestmark = pytest.mark.gpu


def _logits(out, rows):
    import torch
    R, n = rows.H * rows.G, rows.n
    return out["_ws"][: R * n * 4].view(torch.float32).cpu().numpy().reshape(R, n)


def _run(torch, fw, rows, ks, shift=0):
    """Calls dense_topk; shift > 0 moves q, k and v off 16-byte alignment."""
    dev = fw.upload(rows)
    for name in ("q", "k", "v"):
        t = dev[name]
        flat = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
        dev[name] = flat[shift:].view(t.shape).copy_(t)
    out = fw.dense_topk(dev["q"], dev["k"], dev["v"], ks, dev["scale"], dev["bias"])
    torch.cuda.synchronize()
    return out, _logits(out, rows)


@pytest.mark.parametrize("dtype,G,n,d,ks,shift", [
    ("bf16", 1, 33, 128, (1, 32), 0),             # one row, one key past a block
    ("bf16", 4, 5003, 128, (128, 512, 1024), 0),  # few rows: sixteen key splits, sixteen-wave selection
    ("bf16", 17, 1000, 256, (3, 999, 40), 0),     # two row tiles, two column slices
    ("bf16", 65, 95, 72, (90,), 0),               # five row tiles, a partial slice
    ("bf16", 5, 300, 100, (7, 150), 0),           # d no multiple of 8: element loads
    ("bf16", 6, 301, 64, (7, 150), 1),            # unaligned operands
    ("bf16", 3, 200, 160, tuple(range(5, 45, 5)), 0),  # eight budgets, three slices of 64
    ("bf16", 18, 333, 140, (4, 40, 200), 1),      # three budgets in slices of 64, chunks at odd addresses
    ("f32", 9, 290, 104, (4, 40, 200), 0),        # the same on float32, 16-byte loads
    ("f32", 1, 1, 1, (1,), 0),
    ("f32", 16, 64, 64, (16, 64), 0),
    ("f32", 90, 1999, 64, (64, 250, 999), 0),
    ("f32", 7, 257, 200, (1, 2, 3, 4, 250), 0),   # five budgets, four slices
    ("f32", 7, 130, 36, (60, 2), 3),              # d no multiple of 8, unaligned
    ("f32", 33, 2049, 130, (2048, 5), 0),         # element loads, two slices of 128
])
def test_shapes(torch_fw, dtype, G, n, d, ks, shift):
    torch, fw = torch_fw
    rows = W.sink_rows(71, n + G, 2, G, n, d, dtype, sink=4.0)
    out, zg = _run(torch, fw, rows, ks, shift)
    _compare(rows, ks, out, _oracle_rows(rows, ks), torch, zg)


@pytest.mark.parametrize("n", [8193, 32768, 32769])
def test_long_rows_select(torch_fw, n):
    """The selection's limits: 32 logits per thread of 256 and of 1024, and
    rows past them, which are read three times."""
    torch, fw = torch_fw
    rows = W.sink_rows(72, n, 1, 3, n, 32, "bf16", sink=4.0)
    ks = (1024, 5)
    out, zg = _run(torch, fw, rows, ks)
    _compare(rows, ks, out, _oracle_rows(rows, ks), torch, zg)


@pytest.mark.parametrize("H,n,ks", [
    (32, 2100, (9, 500)),    # a row per CU: 16 waves
    (33, 2100, (9, 500)),    # past that four, 32 logits per thread
    (97, 8300, (1000, 3)),   # past 768 rows four waves read them again
    (97, 9300, (1024, 3)),   # 16 with a long index list
])
def test_many_rows_select(torch_fw, H, n, ks):
    """The selection's waves by rows, length and list: the rank order of the
    GPU's own logits, and the largest budget's dropped mass."""
    torch, fw = torch_fw
    rows = W.sink_rows(75, H, H, 8, n, 8, "f32", sink=4.0)
    out, zg = _run(torch, fw, rows, ks)
    want = np.argsort(-zg, axis=1, kind="stable")[:, :max(ks)]
    assert np.array_equal(t2np(out["topk_idx"]).reshape(H * 8, -1), want)
    p = np.exp(zg.astype(np.float64) - zg.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    kept = np.take_along_axis(p, want, axis=1).sum(axis=1)
    t = int(np.argmax(ks))
    assert np.allclose(t2np(out["dropped"])[t].reshape(-1), 1.0 - kept, rtol=1e-4, atol=1e-6)


@pytest.mark.parametrize("case", ["outlier", "equal", "masked", "lowest"])
def test_selection_falls_back(torch_fw, case):
    """Rows whose histogram puts more logits into one bin than rank counting
    takes: a far outlier, all logits equal, and masked keys within the kept
    set (-inf and float32's lowest value)."""
    torch, fw = torch_fw
    n, ks = 1500, (3, 700, 1200)
    rows = W.sink_rows(73, 5, 1, 4, n, 64, "f32", sink=0.0)
    bias = np.zeros(n, np.float32)
    if case == "outlier":
        bias[11] = 3000.0
    elif case == "equal":
        rows.q[:] = 0.0
    else:
        bias[600:] = -np.inf if case == "masked" else np.finfo(np.float32).min
    rows.bias = bias
    out, zg = _run(torch, fw, rows, ks)
    idx = t2np(out["topk_idx"])
    for r in range(4):
        want = np.lexsort((np.arange(n), -zg[r].astype(np.float64)))[:max(ks)]
        assert np.array_equal(idx[0, r], want), (case, r)
    assert np.all(np.isfinite(t2np(out["o"])))
    assert np.all(t2np(out["dropped"]) >= 0.0)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_values_that_are_not_finite(torch_fw, dtype):
    """An infinite value reaches only the sets that hold its key: outputs of
    the other sets equal those without it."""
    torch, fw = torch_fw
    n, ks = 500, (20, 100)
    rows = W.sink_rows(74, 6, 1, 5, n, 128, dtype, sink=4.0)
    clean, zg = _run(torch, fw, rows, ks)
    # the lowest-ranked key of row 0: outside every kept set of that row
    last = int(np.argmin(zg[0]))
    rows.v[0, last, 7] = 0x7F80 if dtype == "bf16" else np.inf
    out, _ = _run(torch, fw, rows, ks)
    outside = [r for r in range(5) if last not in set(t2np(clean["topk_idx"])[0, r].tolist())]
    assert 0 in outside
    a, b = t2np(clean["o_s"]), t2np(out["o_s"])
    assert np.all(np.isfinite(b[:, 0, outside]))
    # the same sums in another order: float32 sums of at most 100 weights
    assert np.allclose(a[:, 0, outside], b[:, 0, outside], rtol=0, atol=1e-5)
    assert np.all(np.isinf(t2np(out["o"])[0, :, 7]))
    cols = np.arange(128) != 7
    assert np.allclose(t2np(clean["o"])[0][:, cols], t2np(out["o"])[0][:, cols], rtol=0, atol=1e-5)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,n", [(1, 300), (1, 4999), (600, 40)])  # one key range, several, one per workgroup
def test_large_values_and_many_keys(torch_fw, dtype, H, n):
    """Values near float32's largest over keys of nearly equal weight: the
    outputs are means of values, so they are finite, and sums of the weights
    unscaled would not be."""
    torch, fw = torch_fw
    rows = W.sink_rows(76, n, H, 3, n, 64, dtype, sink=0.0)
    rows.q[:] = 0
    mag = np.float32(1.5 * 2.0 ** 126)
    rows.v[:] = W.bf16_bits(np.full(rows.v.shape, mag, np.float32)) if dtype == "bf16" else mag
    rows.v[:, ::2, 1] = rows.v[0, 0, 0] ^ 0x8000 if dtype == "bf16" else -mag
    out, _ = _run(torch, fw, rows, (n // 4, n // 2))
    o, o_s = t2np(out["o"]), t2np(out["o_s"])
    # a sum of at most n weights, each of the tier's masses with it: 2 n roundings
    tol = 2 * n * 2.0 ** -24
    cols = np.arange(64) != 1
    assert np.all(np.abs(o[..., cols] / mag - 1) <= tol) and np.all(np.abs(o_s[..., cols] / mag - 1) <= tol)
    assert np.all(np.abs(o[..., 1] / mag + (n % 2) / n) <= tol)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_not_a_number_in_a_row_reaches_all_its_outputs(torch_fw, dtype):
    """A NaN query element: its row has no weights, so every output of that
    row but the indices is NaN; the other rows keep their bits."""
    torch, fw = torch_fw
    n, ks = 700, (3, 90)
    rows = W.sink_rows(77, 4, 1, 6, n, 64, dtype, sink=4.0)
    clean, _ = _run(torch, fw, rows, ks)
    rows.q[0, 2, 5] = 0x7FC0 if dtype == "bf16" else np.nan
    out, _ = _run(torch, fw, rows, ks)
    others = [0, 1, 3, 4, 5]
    assert np.all(np.isnan(t2np(out["o"])[0, 2])) and np.all(np.isnan(t2np(out["o_s"])[:, 0, 2]))
    assert np.all(np.isnan(t2np(out["dropped"])[:, 0, 2]))
    idx = t2np(out["topk_idx"])
    assert idx.min() >= 0 and idx.max() < n
    assert torch.equal(out["o"][:, others], clean["o"][:, others])
    for name in ("o_s", "gap", "dropped"):
        assert torch.equal(out[name][:, :, others], clean[name][:, :, others]), name


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,d", [(33, 128), (1, 64), (70, 256), (2053, 72)])
def test_values_behind_the_last_unit_are_not_read(torch_fw, dtype, n, d):
    """A last block of fewer than seven keys: what lies behind the values of
    the last unit changes no bit of the outputs (a NaN read there would send
    the wave's sums to the key-by-key form, in another order)."""
    torch, fw = torch_fw
    rows = W.sink_rows(75, n, 2, 5, n, d, dtype, sink=4.0)
    dev = fw.upload(rows)
    size = dev["v"].numel()
    got = []
    for fill in (0.0, float("nan")):
        flat = torch.full((size + 64 * d,), fill, dtype=dev["v"].dtype, device="cuda")
        v = flat[:size].view(dev["v"].shape).copy_(dev["v"])
        got.append(fw.dense_topk(dev["q"], dev["k"], v, sorted({1, (n + 2) // 3, n}), dev["scale"], dev["bias"]))
    for name in ("o", "o_s", "gap", "dropped", "topk_idx"):
        assert torch.equal(got[0][name], got[1][name]), name


def test_noalloc_near_its_limit(torch_fw):
    """A call whose logits nearly fill the static scratch array still runs
    there (with fewer key splits), and gives what the workspace call gives."""
    torch, fw = torch_fw
    n, G = 64 * 1024, 250  # 62.5 MiB of logits
    g = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn((1, G, 64), generator=g, device="cuda").bfloat16()
    k = torch.randn((1, n, 64), generator=g, device="cuda").bfloat16()
    v = torch.randn((1, n, 64), generator=g, device="cuda").bfloat16()
    a = fw.dense_topk(q, k, v, (64,), want_idx=False)
    b = fw.dense_topk_noalloc(q, k, v, (64,), want_idx=False)
    for name in ("o", "o_s", "gap", "dropped"):
        assert torch.equal(a[name], b[name]), name
