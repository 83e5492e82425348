"""The launch that opens a forward (first RMSNorm and rotary table together; it also writes the
residual stream where the input is the embeddings) and the register-resident norm at every vector
width: hidden sizes of 1, 2, 3, 5, 6, 7 (the general kernel), 8 and 10 times 256, two layers and
the final norm against the oracle, fp32 at 1e-4 and bf16 (bf16 rows in, fp16 out) at 3e-2; and
encode_layers, whose first output projection reads the input rows as its residual, in place, out
of place and on buffers aligned like one float only, bit for bit the same."""
import sys

import numpy as np
import pytest

from oracle import te_oracle as O
from synth import workloads as W
from tests.gpu_common import layout_tuples, make_encoder, oracle_encode, rel_err

pytestmark = pytest.mark.gpu

LAYOUTS = (W.SeqLayout(2, 1, 3, 4, 5), W.SeqLayout(0, 0, 0, 0, 1), W.SeqLayout(0, 1, 4, 4, 16))


@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 7, 10, 12])
def test_norm_widths_bf16(n):
    import torch
    from paper_2606_05981_amd.encoder import build_positions
    assert torch.cuda.is_available(), "no GPU"
    dims = W.DIMS_TINY.with_(hidden=256 * n, ffn=256, dtype="bf16")
    emb = W.embeddings(dims, LAYOUTS)
    print("hidden", dims.hidden, file=sys.stderr, flush=True)
    enc = make_encoder(dims, max_tokens=64, max_batch=4, max_seq=64)
    out = enc.encode(torch.from_numpy(emb).to("cuda", torch.bfloat16), build_positions(layout_tuples(LAYOUTS)),
                     W.seq_lens(LAYOUTS))
    torch.cuda.synchronize()
    enc.close()
    err = rel_err(out.cpu().numpy(), oracle_encode(dims, emb, LAYOUTS))
    print("  err", err, file=sys.stderr, flush=True)
    assert err <= 3e-2


@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 7, 8, 10])
def test_norm_widths(n):
    import torch
    from paper_2606_05981_amd.encoder import build_positions
    assert torch.cuda.is_available(), "no GPU"
    dims = W.DIMS_TINY.with_(hidden=256 * n, ffn=256)
    emb = W.embeddings(dims, LAYOUTS)
    print("hidden", dims.hidden, file=sys.stderr, flush=True)
    enc = make_encoder(dims, max_tokens=64, max_batch=4, max_seq=64)
    out = enc.encode(torch.from_numpy(emb).cuda(), build_positions(layout_tuples(LAYOUTS)), W.seq_lens(LAYOUTS))
    torch.cuda.synchronize()
    enc.close()
    assert rel_err(out.cpu().numpy(), oracle_encode(dims, emb, LAYOUTS)) <= 1e-4


@pytest.mark.parametrize("dims", [W.DIMS_TINY, W.DIMS_FULL.with_(n_layers=2)], ids=["fp32", "bf16"])
def test_residual_stream_buffers(dims):
    import torch
    from paper_2606_05981_amd.encoder import build_positions
    assert torch.cuda.is_available(), "no GPU"
    lens = W.seq_lens(LAYOUTS)
    T, D = sum(lens), dims.hidden
    x = torch.from_numpy(np.random.default_rng(3).standard_normal((T, D), dtype=np.float32)).cuda()
    enc = make_encoder(dims, max_tokens=64, max_batch=4, max_seq=64)
    pos = build_positions(layout_tuples(LAYOUTS))

    def shifted():
        return torch.zeros(T * D + 1, device="cuda")[1:].view(T, D)   # 4-byte aligned

    for l0, l1 in ((0, 2), (1, 2), (1, 1)):
        print("layers", l0, l1, file=sys.stderr, flush=True)
        ref = enc.encode_layers(x, pos, lens, l0, l1)
        inplace = x.clone()
        enc.encode_layers(inplace, pos, lens, l0, l1, h_out=inplace)
        src, dst = shifted(), shifted()
        src.copy_(x)
        keep = src.clone()
        enc.encode_layers(src, pos, lens, l0, l1, h_out=dst)
        torch.cuda.synchronize()
        assert torch.equal(ref, inplace) and torch.equal(ref, dst)
        assert torch.equal(src, keep)
    enc.close()


@pytest.mark.parametrize("dims,fmt,lens", [
    (W.DIMS_TINY, 0, (64, 33)), (W.DIMS_FULL.with_(n_layers=2), 0, (320, 17, 300)),
    (W.DIMS_FULL.with_(n_layers=2), 1, (320, 257)), (W.DIMS_FULL.with_(n_layers=2), 1, (1,)),
], ids=["fp32_97", "bf16_637", "e4m3_577", "e4m3_1"])
def test_residual_read_from_input(dims, fmt, lens):
    """The first layer's output projection (whole or split over K) reads the input rows and writes
    every element of h_out: the result equals the in-place one bit for bit, whatever h_out held."""
    import torch
    from paper_2606_05981_amd.encoder import build_positions
    assert torch.cuda.is_available(), "no GPU"
    T, D = sum(lens), dims.hidden
    x = torch.from_numpy(np.random.default_rng(5).standard_normal((T, D), dtype=np.float32)).cuda()
    keep = x.clone()
    enc = make_encoder(dims, max_tokens=640, max_batch=4, max_seq=320, weight_format=fmt)
    pos = build_positions([(n, 0, 0, 0, 0) for n in lens])
    for l0, l1 in ((0, 1), (0, 2), (1, 2)):
        print(T, "rows, layers", l0, l1, file=sys.stderr, flush=True)
        inplace = x.clone()
        enc.encode_layers(inplace, pos, list(lens), l0, l1, h_out=inplace)
        out = torch.full_like(x, float("nan"))
        enc.encode_layers(x, pos, list(lens), l0, l1, h_out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, inplace) and torch.equal(x, keep)
    enc.close()
