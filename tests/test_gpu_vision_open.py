"""The launch that opens the vision tower (patch extraction and rotary table): patch sizes read
eight pixels at a time and one at a time, non-square images, both storage types, pixels aligned
like one element only. One block and the merger against the oracle: fp32 at 1e-4, bf16 at 1e-2
(max|gpu - oracle| / rms, the bars of the vision parity tests); the unaligned copy bit for bit."""
import sys

import pytest

from oracle import vit_oracle as V
from synth import vision as SV
from tests.gpu_common import rel_err

pytestmark = pytest.mark.gpu

CASES = {  # patch, channels: values per patch a multiple of 64
    "patch4": dict(patch=4, in_channels=4),
    "patch8": dict(patch=8, in_channels=1),
    "patch16_merge1": dict(patch=16, in_channels=3, merge=1),
    "patch24": dict(patch=24, in_channels=1),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_patch_sizes(case, dtype):
    import torch
    from paper_2606_05981_amd import binding as B
    from paper_2606_05981_amd.encoder import VisionEncoder
    assert torch.cuda.is_available(), "no GPU"
    v = SV.VDIMS_TINY.with_(depth=1, dtype=dtype, **CASES[case])
    s = v.patch * v.merge
    h, w = 3 * s, 5 * s
    img = SV.images(v, 2, h, w)
    print("vision open", case, dtype, h, w, file=sys.stderr, flush=True)
    bf = dtype == "bf16"
    cfg = B.make_vision_config(v.depth, v.hidden, v.n_heads, v.head_dim, v.ffn, patch=v.patch, merge=v.merge,
                               in_channels=v.in_channels, out_hidden=v.out_hidden, ln_eps=v.ln_eps,
                               rope_theta=v.rope_theta, dtype=B.MTE_BF16 if bf else B.MTE_F32, out_dtype=B.MTE_F32,
                               max_images=2, max_side=w)
    enc = VisionEncoder.from_host(cfg, SV.outer_weights(v), [SV.block_weights(v, 0)])
    px = torch.from_numpy(img).to("cuda", torch.bfloat16 if bf else torch.float32)
    out = enc.encode(px)
    odd = torch.zeros(px.numel() + 1, dtype=px.dtype, device="cuda")[1:].view(px.shape)
    odd.copy_(px)
    out2 = enc.encode(odd)
    torch.cuda.synchronize()
    enc.close()
    ref = V.encode(img, v, lambda l: SV.block_weights(v, l), SV.outer_weights(v))
    assert rel_err(out.cpu().numpy(), ref) <= (1e-2 if bf else 1e-4)
    assert torch.equal(out, out2)
