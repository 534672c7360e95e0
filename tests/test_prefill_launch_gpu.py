"""The prefill's launches against the fp64 oracle where their shape changes:
all layers in one launch (groups of layers sharing heads, several heads per
layer, maps given as tables), the token-split form of small grids, row blocks
of head dim 128, and every form with references that rise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from gpu_util import check_close, f64, prefill_rounding_bound, say  # noqa: E402
from test_prefill_gpu import PrefillCase, _check_case, _gpu, mlkv  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l,h,m,g,D,B,T,ctx", [
    (6, 12, 2, 3, 64, 2, 33, [0, 31]),     # three layers share three heads each
    (4, 5, 2, 5, 64, 3, 50, [7, 0, 64]),   # one row per head and layer: two per token
    (6, 4, 1, 2, 128, 2, 41, [30, 1]),     # six layers on one group, head dim 128
])
def test_all_layers_in_one_launch(l, h, m, g, D, B, T, ctx):
    w = synth.Workload("all_layers", l=l, h=h, m=m, g=g, D=D, B=B, ctx=max(ctx), T=T, seed=301)
    tag = f"all layers l{l} h{h} m{m} g{g} D{D} B{B} T{T}"
    say(tag)
    _check_case(PrefillCase(w, ctx=ctx), tag)


@pytest.mark.parametrize("kv_of,owner_of", [
    ([[0] * 4, [0] * 4, [1] * 4, [1] * 4], [0, 2]),  # equal groups: one launch
    ([[0] * 4, [1] * 4, [0] * 4, [1] * 4], [0, 1]),  # interleaved: layer by layer
    ([[0, 0, 1, 1], [0, 0, 1, 1], [1] * 4, [0] * 4], [0, 0]),  # part of a group
])
def test_table_maps(kv_of, owner_of):
    kv_of, owner_of = np.array(kv_of, np.int32), np.array(owner_of, np.int32)
    w = synth.Workload("tables", l=4, h=4, m=2, g=1, D=64, B=2, ctx=40, T=37, seed=302)
    tag = f"prefill tables {kv_of.tolist()}"
    say(tag)
    _check_case(PrefillCase(w, ctx=[3, 40], kv_of=kv_of, owner_of=owner_of), tag)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,ctx", [
    (1, [0, 255]),     # one row block, fewer tiles than waves
    (9, [223, 224]),   # last tile full and one past it
    (40, [511, 3]),    # waves without a tile beside waves with several
])
def test_token_split_form(D, T, ctx):
    w = synth.Workload("split", l=2, h=6, m=2, g=2, D=D, B=2, ctx=max(ctx), T=T, k_scale=3.0,
                       seed=303)
    tag = f"prefill split D{D} T{T} ctx{ctx}"
    say(tag)
    _check_case(PrefillCase(w, ctx=ctx), tag)


@pytest.mark.parametrize("B,T,ctx", [
    (10, 102, 0),    # 64-row workgroups, the last one ragged
    (16, 130, 33),   # several a compute unit, cached prefix
    (17, 121, 0),    # blocks that start inside a token's heads
])
def test_head_dim_128_row_blocks(B, T, ctx):
    w = synth.Workload("rows128", l=1, h=64, m=1, g=4, D=128, B=B, ctx=ctx, T=T, seed=304)
    tag = f"prefill D128 B{B} T{T} ctx{ctx}"
    say(tag)
    _check_case(PrefillCase(w), tag)


class RisingCase(PrefillCase):
    """Keys that grow from tile to tile, so that a row's maximum keeps moving
    far past the reference its first tile set; ragged contexts, poisoned tails."""

    def __init__(self, w):
        top = w.ctx
        super().__init__(w, ctx=[top - (37 * b) % (top + 1) for b in range(w.B)])
        h = self.host
        tile = np.arange(self.S) // 32
        growth = (1 + 0.75 * tile).astype(np.float32)[:, None]
        for b, c in enumerate(h["ctx"]):
            rows = synth.bf16_to_f32(h["k_cache"][:, b, :c]) * growth[:c]
            h["k_cache"][:, b, :c] = synth.f32_to_bf16(rows)
            rows = synth.bf16_to_f32(h["k_new"][b]) * growth[c:c + w.T, None]
            h["k_new"][b] = synth.f32_to_bf16(rows)
        self.cache.load_rows(h["k_cache"], h["v_cache"])
        self.k_new = mlkv.bf16_tensor(h["k_new"], "cuda")


@pytest.mark.parametrize("form,l,h,m,g,D,B,T,top", [
    ("plain", 4, 8, 2, 4, 64, 24, 50, 110),
    ("plain", 4, 8, 2, 4, 128, 24, 50, 110),
    ("wide", 6, 12, 3, 4, 128, 43, 33, 287),
    ("split", 2, 12, 2, 1, 64, 2, 80, 464),
    ("split", 2, 12, 2, 1, 128, 2, 80, 464),
])
def test_references_rise_in_every_form(form, l, h, m, g, D, B, T, top):
    """Each form of the prefill at a grid that takes it (the host driver of
    test_sanitizers.py holds the choice at these sizes), layers sharing heads,
    several heads a layer, rows whose scores leave the first reference by more
    than any form's slack (2^8 a weight, 2^12 a sum), and bit-for-bit repeats."""
    w = synth.Workload("rising", l=l, h=h, m=m, g=g, D=D, B=B, ctx=top, T=T, k_scale=2.0, seed=305)
    tag = f"prefill {form} rising l{l} D{D} B{B} T{T}"
    say(tag)
    c = RisingCase(w)
    out = c.run().cpu().numpy()
    say(tag + " again")
    for _ in range(3):
        assert np.array_equal(c.run().cpu().numpy().view(np.uint32), out.view(np.uint32)), tag
    k_gpu, v_gpu = c.read_cache()
    sel = sorted({0, 1, B // 2, B - 1})  # the oracle takes these sequences
    host = c.host
    k, v = (np.ascontiguousarray(host[n][:, sel]) for n in ("k_cache", "v_cache"))
    q, ctx = np.ascontiguousarray(host["q"][:, sel]), host["ctx"][sel]
    ref = oracle.prefill_step(q, k, v, host["k_new"][sel], host["v_new"][sel], c.kv_of, c.owner_of,
                              ctx)
    assert np.array_equal(k_gpu[:, sel], k) and np.array_equal(v_gpu[:, sel], v), f"{tag}: cache"
    L = int(ctx[0]) + T
    x = f64(q[0, 0, -1]) @ f64(k[c.kv_of[0, 0], 0, :L]).T * (np.log2(np.e) / np.sqrt(D))
    assert (x.max(axis=1) - x[:, :32].max(axis=1)).max() > 13  # the last token's rows
    check_close(out[:, sel], ref, tag, bound=prefill_rounding_bound(q, k, v, c.kv_of, ctx, ref))
