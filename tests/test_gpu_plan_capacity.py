"""The launch plan depends on the batch's tokens and the model shape, not on how large a workspace
the encoder was created with: the same batch through encoders of different max_tokens is the same
bit for bit. Widest product = the QKV projection, whose partial sums are then what the workspace
is sized for, at row counts where splitting K by eight fits only the larger workspace."""
import sys

import numpy as np
import pytest

from synth import workloads as W
from tests.gpu_common import make_encoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    W.Dims(n_layers=1, hidden=4096, n_q_heads=16, n_kv_heads=8, head_dim=128, ffn=256, dtype="f32"),
    W.Dims(n_layers=1, hidden=1024, n_q_heads=8, n_kv_heads=4, head_dim=128, ffn=512, dtype="f32"),
    W.Dims(n_layers=1, hidden=2048, n_q_heads=16, n_kv_heads=8, head_dim=128, ffn=1024),
], ids=["f32_4096", "f32_1024", "bf16_2048"])
def test_plan_ignores_capacity(dims):
    import torch
    from paper_2606_05981_amd.encoder import build_positions
    assert torch.cuda.is_available(), "no GPU"
    small = make_encoder(dims, max_tokens=520, max_batch=2, max_seq=400)
    large = make_encoder(dims, max_tokens=4096, max_batch=2, max_seq=400)
    for lens in ((257,), (150, 150), (400,), (256, 256)):
        print(dims.hidden, lens, file=sys.stderr, flush=True)
        T = sum(lens)
        x = torch.from_numpy(np.random.default_rng(T).standard_normal((T, dims.hidden), dtype=np.float32)).cuda()
        pos = build_positions([(n, 0, 0, 0, 0) for n in lens])
        a = small.encode_layers(x, pos, list(lens), 0, 1)
        b = large.encode_layers(x, pos, list(lens), 0, 1)
        torch.cuda.synchronize()
        assert torch.equal(a, b), lens
    small.close()
    large.close()
