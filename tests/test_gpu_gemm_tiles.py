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


@pytest.mark.parametrize("rows", [1, 31, 33, 65, 129, 700])
def test_fp32_rows(rows):
    x, pos, lens, got = run_layer(TINY, rows)
    ref = O.layer_forward(x, pos, lens, layer_w(TINY, 0), TINY)
    assert rel_err(got, ref) <= 1e-4
