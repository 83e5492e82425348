"""One decoder layer at row counts around the edges of the projection GEMMs' tiles: every row
count takes its own tiles and K splits (the planner weighs whole rounds of workgroups), the last
tile of each product is partly or almost wholly past the batch, and the V^T tiles of the QKV
epilogue end in either half of their 32 tokens. The sequences are packed so that the total is the
row count. bf16 at the per-layer bar 1e-2, e4m3 weights against the oracle on the dequantised
weights at the same bar, fp32 (tiny shape) at 1e-4: max|gpu - oracle| / rms, the bars the parity
tests hold everywhere."""
import sys

import numpy as np
import pytest

from oracle import te_oracle as O
from synth import workloads as W
from tests.gpu_common import layer_w, layer_w_e4m3, layout_tuples, make_encoder, rel_err

pytestmark = pytest.mark.gpu

FULL = W.DIMS_FULL.with_(n_layers=1)
TINY = W.DIMS_TINY.with_(n_layers=1)


def layouts_for(rows):
    """Text sequences of at most 97 tokens (odd, so that most start inside a tile) with `rows`
    tokens in all."""
    lens = [97] * (rows // 97) + ([rows % 97] if rows % 97 else [])
    return tuple(W.SeqLayout(0, 0, 0, 0, n) for n in lens)


def run_layer(dims, rows, **kw):
    import torch
    from paper_2606_05981_amd.encoder import build_positions
    assert torch.cuda.is_available(), "no GPU"
    lay = layouts_for(rows)
    lens = W.seq_lens(lay)
    print("rows", rows, kw, file=sys.stderr, flush=True)
    # residual streams of the size they have inside a stack (the embeddings' 0.02 would hide
    # the norm's epsilon and leave the update alone)
    x = np.random.default_rng(rows).standard_normal((rows, dims.hidden), dtype=np.float32)
    enc = make_encoder(dims, max_tokens=rows, max_batch=len(lens), max_seq=97, **kw)
    h = enc.encode_layers(torch.from_numpy(x).cuda(), build_positions(layout_tuples(lay)), lens, 0, 1)
    torch.cuda.synchronize()
    enc.close()
    return x, O.positions(lay), lens, h.cpu().numpy()


@pytest.mark.parametrize("rows", [1, 17, 31, 33, 65, 97, 129, 161, 225, 257, 337, 513, 769, 1153, 1537, 2049, 2600])
def test_bf16_rows(rows):
    x, pos, lens, got = run_layer(FULL, rows)
    ref = O.layer_forward(x, pos, lens, layer_w(FULL, 0), FULL)
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= 1e-2


@pytest.mark.parametrize("rows", [17, 33, 97, 225, 513])
def test_e4m3_rows(rows):
    x, pos, lens, got = run_layer(FULL, rows, weight_format=1)
    ref = O.layer_forward(x, pos, lens, layer_w_e4m3(FULL, 0), FULL)
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= 1e-2


@pytest.mark.parametrize("rows", [769, 1153, 1537, 2049, 2600])
def test_e4m3_many_rows(rows):
    """The e4m3 plans of large batches: whole products on the 96- to 192-row tiles, the down
    projection split by two at 769 rows."""
    x, pos, lens, got = run_layer(FULL, rows, weight_format=1)
    ref = O.layer_forward(x, pos, lens, layer_w_e4m3(FULL, 0), FULL)
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= 1e-2


@pytest.mark.parametrize("rows", [129, 769, 1153, 2049])
def test_half_heads_without_qk_norm(rows):
    """The QKV epilogue with half a 128-wide head per wave (32x128, 128x128, 192x128 and 160x256
    tiles) and no QK-norm: rotation and operand layout without the exchange of the sums."""
    dims = FULL.with_(qk_norm=0)
    x, pos, lens, got = run_layer(dims, rows)
    ref = O.layer_forward(x, pos, lens, layer_w(dims, 0), dims)
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= 1e-2


@pytest.mark.parametrize("rows", [1, 31, 33, 65, 129, 700])
def test_fp32_rows(rows):
    x, pos, lens, got = run_layer(TINY, rows)
    ref = O.layer_forward(x, pos, lens, layer_w(TINY, 0), TINY)
    assert rel_err(got, ref) <= 1e-4


WIDE_F32 = W.Dims(n_layers=1, hidden=1024, n_q_heads=8, n_kv_heads=4, head_dim=128, ffn=3072, dtype="f32")


@pytest.mark.parametrize("rows,qk_norm", [(1, 1), (33, 1), (161, 1), (257, 1), (400, 0), (400, 1), (513, 1),
                                          (769, 1), (1537, 1), (2049, 0), (2049, 1)])
def test_wide_fp32_rows(rows, qk_norm):
    """fp32 at width 1024, heads of 128: the eight-wave tiles (192, 128 and 96 rows) and 32x128,
    whole and split over K, whose QKV epilogue halves a head between two waves."""
    dims = WIDE_F32.with_(qk_norm=qk_norm)
    x, pos, lens, got = run_layer(dims, rows)
    assert rel_err(got, O.layer_forward(x, pos, lens, layer_w(dims, 0), dims)) <= 1e-4


@pytest.mark.parametrize("rows", [1025, 1537, 2049])
def test_tiny_fp32_many_rows(rows):
    """fp32 heads of 64 on the tiles of many rows (32x128, 96x128, 128x128, 128x64)."""
    x, pos, lens, got = run_layer(TINY, rows)
    assert rel_err(got, O.layer_forward(x, pos, lens, layer_w(TINY, 0), TINY)) <= 1e-4


@pytest.mark.parametrize("lens,bar", [((32,), 4.1e-7), ((128, 128), 4.75e-7), ((320, 192), 5.3e-7),
                                      ((320,) * 4, 6.0e-7)])
def test_fp32_sums_in_stages(lens, bar):
    """The fp32 products sum K in stages of 32: the relative error of two layers and the final norm
    against float64, averaged over four inputs, stays below the geometric middle of what the
    kernels measure with stages and with one chain over each K range (same tiles and splits):
    3.58e-7 and 4.76e-7 at 32 tokens, 4.07e-7 and 5.60e-7 at 2 x 128, 4.30e-7 and 6.58e-7 at
    320 + 192, 4.39e-7 and 8.28e-7 at 4 x 320. Averages over other inputs differ by 0.2e-7."""
    import torch
    from perf import cases as C
    case = dict(kind="encode", lens=",".join(map(str, lens)), layers=2, dtype="f32", weights="dtype", qk_norm=1,
                layout=0, prefix=0)
    errs = []
    for seed in range(1, 5):
        s = C.prepare(case, seed)
        got, ref = C.run(s)["hidden"].double(), C.exact(case, seed)["hidden"]
        errs.append(((got - ref).norm() / ref.norm()).item())
        torch.cuda.synchronize()
        s["enc"].close()
    assert sum(errs) / len(errs) <= bar, errs
