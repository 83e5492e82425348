"""The tile table of the projection GEMMs (csrc/gemm_kernel.h), read as text: what the planner and
the launches assume of every tile, no GPU needed. The LDS ring fits 160 KB per CU; no modelled
cost of a K stage is below the time its MFMAs take at the card's clock limit (the fp32 products
were once planned with the fp16 costs, a quarter of that time); and every shape the encoders
accept has a tile in every mode."""
import os
import re

import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_05981_amd", "csrc",
                      "gemm_kernel.h")
MODES = ("f32", "f16", "f8w")
STAGE_BYTES = 128


def tiles():
    out = []
    with open(HEADER) as f:
        for m in re.finditer(r"^  X\(([^)]*)\)", f.read(), re.M):
            v = [float(x) for x in m.group(1).split(",")]
            assert len(v) == 15, m.group(0)
            bm, bn, wm, wn, p, occ, f32, w8 = (int(x) for x in v[1:9])
            out.append(dict(id=int(v[0]), bm=bm, bn=bn, wm=wm, wn=wn, p=p, occ=occ,
                            built={"f32": f32, "f16": 1, "f8w": w8},
                            stage={"f16": v[9], "f8w": v[11], "f32": v[13]},
                            tile={"f16": v[10], "f8w": v[12], "f32": v[14]}))
    return out


def test_ids_and_waves():
    ts = tiles()
    assert [t["id"] for t in ts] == list(range(len(ts))) and len(ts) > 1
    for t in ts:
        assert t["wm"] * t["wn"] in (4, 6, 8) and t["bm"] % 32 == 0
        assert t["bm"] % (16 * t["wm"]) == 0 and t["bn"] % (16 * t["wn"]) == 0


@pytest.mark.parametrize("mode", MODES)
def test_lds_ring_fits(mode):
    for t in tiles():
        if t["built"][mode]:
            w = t["bn"] // 2 if mode == "f8w" else t["bn"]
            assert t["p"] * (t["bm"] + w) * STAGE_BYTES * t["occ"] <= 160 * 1024, t


@pytest.mark.parametrize("mode", MODES)
def test_costs_are_above_the_mfma_time(mode):
    # flop per cycle and CU: 256 CUs at 2.4 GHz give 2.5 PFLOP/s dense in fp16, 157 TFLOP/s in fp32
    rate = {"f32": 256, "f16": 4096, "f8w": 4096}[mode] * 2.4e9
    k = STAGE_BYTES // (4 if mode == "f32" else 2)
    for t in tiles():
        if t["built"][mode]:
            floor = 2.0 * t["bm"] * t["bn"] * k / rate * 1e6
            # two workgroups share a CU: each alone on it, the cost the model scales
            assert t["stage"][mode] >= floor and t["tile"][mode] > 0, (t, floor)


def fits(t, mode, n, epi, head_dim=None):
    if not t["built"][mode] or n % t["bn"]:
        return False
    cols = t["bn"] // t["wn"]
    if epi == "swiglu":
        return cols % 32 == 0
    if epi == "qkv":
        return cols % head_dim == 0 or (head_dim == 128 and cols == 64 and t["wn"] % 2 == 0)
    return True


def has_tile(mode, n, epi, head_dim=None):
    return any(fits(t, mode, n, epi, head_dim) for t in tiles())


@pytest.mark.parametrize("mode", MODES)
def test_every_text_width_has_a_tile(mode):
    for n in range(256, 4096 + 1, 256):                      # hidden; 2 x ffn in gate/up
        assert has_tile(mode, n, "resid") and has_tile(mode, 2 * n, "swiglu")
    for hd in (64, 128):
        for q in range(256, 4096 + 1, 256):                  # q columns and twice the kv columns
            for kv in range(128, q + 1, 128):
                assert has_tile(mode, q + 2 * kv, "qkv", hd)


@pytest.mark.parametrize("mode", ("f32", "f16"))
def test_every_vision_width_has_a_tile(mode):
    for n in range(64, 4096 + 1, 64):                        # hidden, ffn, output width
        assert has_tile(mode, n, "store") and has_tile(mode, n, "resid") and has_tile(mode, n, "gelu")
        assert has_tile(mode, 3 * n, "qkv", 64)
        if n % 128 == 0:
            assert has_tile(mode, 3 * n, "qkv", 128)
