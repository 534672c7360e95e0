"""The prefill's launches against the fp64 oracle where their shape changes:
all layers in one launch (groups of layers sharing heads, several heads per
layer, maps given as tables), the token-split form of small grids, 64- and
256-row workgroups of head dim 128."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from gpu_util import say  # noqa: E402
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
    (16, 130, 33),   # 256-row workgroups at two per compute unit, ragged, cached prefix
    (17, 121, 0),
])
def test_head_dim_128_row_blocks(B, T, ctx):
    w = synth.Workload("rows128", l=1, h=64, m=1, g=4, D=128, B=B, ctx=ctx, T=T, seed=304)
    tag = f"prefill D128 B{B} T{T} ctx{ctx}"
    say(tag)
    _check_case(PrefillCase(w), tag)
