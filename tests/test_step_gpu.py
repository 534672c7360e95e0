"""The decode step in one launch (csrc/step.hip) against the fp64 oracle and
against the layer-by-layer launches, at the edges of its plan: one to three
blocks of query rows, rows in several chunks, split and whole units, four- and
eight-wave workgroups, and maps given as tables."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from gpu_util import DeviceWorkload, check_close, say, step_rounding_bound  # noqa: E402

pytestmark = pytest.mark.gpu

mlkv = pytest.importorskip("paper_2406_09297_amd")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mlkv.lib()
    yield


def _lengths(B, top):
    """Contexts around tile edges, an empty sequence, the longest."""
    base = [min(x, top) for x in (-1, 0, 30, 31, 32, 33, 63, 64, top)]
    return np.array([base[i % len(base)] if i < len(base) else (i * 37) % (top + 1)
                     for i in range(B)], np.int32)


def _step(dw, out_dtype=torch.float32, ws=None, rd=0):
    w = dw.w  # dw.hint: the caller's bound of the lengths, if any
    out = torch.full((w.l, w.B, w.h, w.D), float("nan"), dtype=out_dtype, device="cuda")
    mlkv.decode_step(dw.q, dw.k_new, dw.v_new, dw.cache, dw.map, dw.ctx, out,
                     max_len_hint=getattr(dw, "hint", 0), ws=dw.ws if ws is None else ws,
                     rotary_dims=rd)
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


def _prepare(l, h, m, g, D, B, top, seed):
    w = synth.Workload("one_launch", l=l, h=h, m=m, g=g, D=D, B=B, ctx=top, seed=seed)
    dw = DeviceWorkload(w)
    ctx = _lengths(B, top)
    dw.host["ctx"] = ctx
    dw.ctx = torch.from_numpy(ctx).cuda()
    return dw


def _check(dw, tag):
    out = _step(dw)
    again = _step(dw)
    assert np.array_equal(out, again), f"{tag}: a repeated step differs"
    k_gpu, v_gpu = dw.read_cache()
    k, v = dw.host["k_cache"].copy(), dw.host["v_cache"].copy()
    ref = oracle.decode_step(dw.host["q"], k, v, dw.host["k_new"], dw.host["v_new"], dw.kv_of,
                             dw.owner_of, dw.host["ctx"])
    assert np.array_equal(k_gpu, k) and np.array_equal(v_gpu, v), f"{tag}: cache differs"
    check_close(out, ref, tag, bound=step_rounding_bound(dw.host["q"], k, v, dw.kv_of,
                                                         dw.host["ctx"], ref))
    return out


@pytest.mark.parametrize("l,h,m,g,D,B,top", [
    (4, 4, 2, 4, 64, 9, 70),       # two rows per KV head; whole units
    (4, 8, 2, 1, 64, 9, 700),      # sixteen rows: one full block; split runs
    (4, 9, 2, 1, 64, 9, 900),      # eighteen rows: two blocks, the second nearly empty
    (6, 12, 2, 1, 64, 9, 1300),    # thirty-six rows in two chunks, split runs
    (12, 12, 1, 1, 64, 2, 2047),   # 144 rows in five chunks, eight runs per unit
    (6, 12, 2, 1, 64, 130, 95),    # 260 units: three blocks on four-wave workgroups
    (12, 12, 1, 1, 64, 60, 95),    # 60 units x 144 rows: three chunks of three blocks
    (4, 2, 4, 2, 64, 100, 40),     # 800 units of at most two tiles: four waves, whole units
    (4, 8, 2, 2, 128, 9, 500),     # head dim 128, eight rows
    (8, 8, 1, 2, 128, 3, 1500),    # 32 rows in two chunks, split runs
    (8, 8, 1, 2, 128, 150, 40),    # 300 units: two blocks on four-wave workgroups
    (8, 16, 1, 1, 128, 40, 70),    # 128 rows: four chunks of two blocks
])
def test_one_launch_step_matches_oracle(l, h, m, g, D, B, top):
    tag = f"one launch l{l} h{h} m{m} g{g} D{D} B{B} top{top}"
    say(tag)
    _check(_prepare(l, h, m, g, D, B, top, seed=31 + l + h), tag)


@pytest.mark.parametrize("l,h,m,g,D,ctx", [
    (32, 32, 2, 2, 128, [1500, 700]),       # 256 rows: eight chunks of two blocks, four runs
    (12, 16, 1, 1, 64, [4200, 1031]),       # 192 rows: four chunks of three blocks, 16 runs
    (8, 12, 1, 1, 128, [4200]),             # 96 rows, 16 runs merged in two rounds
    (2, 8, 1, 1, 64, [33000, 9300, 500]),   # 32 runs, 17 by the second one's length
    (4, 6, 2, 1, 128, [12500]),             # 19 runs of two units
    (2, 4, 2, 2, 128, [33000, 16000]),      # eight units: 16 runs, half of the compute units
])
def test_split_runs_match_oracle(l, h, m, g, D, ctx):
    """Units in several runs at the widest row blocks, in more runs than a
    merge takes at a time, and in fewer than the longest unit's."""
    tag = f"split runs l{l} h{h} m{m} g{g} D{D} ctx{ctx}"
    say(tag)
    dw = _prepare(l, h, m, g, D, len(ctx), max(ctx), seed=53 + l + h)
    dw.host["ctx"] = np.array(ctx, np.int32)
    dw.ctx = torch.from_numpy(dw.host["ctx"]).cuda()
    _check(dw, tag)


@pytest.mark.parametrize("runs", [1, 2, 3, 7])
def test_workspace_for_fewer_runs(runs):
    """A workspace that ends where `runs` runs of each unit end."""
    dw = _prepare(12, 12, 4, 1, 64, 2, 2000, seed=5)
    dw.host["ctx"] = np.array([2000, 1100], np.int32)
    dw.ctx = torch.from_numpy(dw.host["ctx"]).cuda()
    rows = 2 * 4 * 2 * runs * 18  # sequences x KV heads x chunks x runs x rows of a chunk
    size = 65536 * 4 + -(-rows * 64 * 4 // 256) * 256 + rows * 8
    tag = f"workspace for {runs} runs"
    say(tag)
    tight = 65536 * 4 + 60 * 1024  # the layer-by-layer step's needs: at least these
    dw.ws = torch.zeros(max(size, tight), dtype=torch.uint8, device="cuda")
    _check(dw, tag)


@pytest.mark.parametrize("kv_of,owner_of", [
    ([[0] * 4, [0] * 4, [1] * 4, [1] * 4], [0, 2]),              # equal groups: one launch
    ([[0, 0, 1, 1], [2, 2, 3, 3]], [0, 0, 1, 1]),                # no sharing across layers
    ([[0] * 4, [0] * 4, [0] * 4, [1] * 4], [0, 3]),              # groups of different sizes
    ([[0] * 4, [1] * 4, [0] * 4, [1] * 4], [0, 1]),              # groups interleaved
    ([[0, 0, 1, 1], [0, 0, 1, 1], [2] * 4, [2] * 4], [0, 0, 2]),  # head counts differ
    ([[0, 0, 1, 1], [1] * 4], [0, 0]),                           # a layer reading half a group
])
def test_table_maps_match_oracle_and_layer_by_layer(kv_of, owner_of, monkeypatch):
    """Maps that do and do not fall into equal groups of layers: the oracle
    decides, and the layer-by-layer launches (any override of the per-layer
    plan selects them) leave the same cache and outputs within the rounding
    of the softmax weights."""
    kv_of, owner_of = np.array(kv_of, np.int32), np.array(owner_of, np.int32)
    l, n_kv = kv_of.shape[0], owner_of.size
    w = synth.Workload("tables", l=l, h=4, m=n_kv, g=1, D=64, B=9, ctx=330, seed=77) \
        if l % n_kv == 0 else synth.Workload("tables", l=n_kv * l, h=4, m=n_kv, g=1, D=64, B=9,
                                             ctx=330, seed=77)
    dw = DeviceWorkload(w)
    if w.l != l:  # the generator's layers beyond the map's are not used
        dw.host["q"] = np.ascontiguousarray(dw.host["q"][:l])
        dw.q = mlkv.bf16_tensor(dw.host["q"], "cuda")
        dw.w = synth.Workload("tables", l=l, h=4, m=n_kv, g=1, D=64, B=9, ctx=330, seed=77)
    ctx = _lengths(9, 330)
    dw.host["ctx"], dw.ctx = ctx, torch.from_numpy(ctx).cuda()
    dw.map = mlkv.Map.from_tables(kv_of, owner_of)
    dw.kv_of, dw.owner_of = kv_of, owner_of
    dw.ws = mlkv.workspace(dw.map, 9, dw.S, 64)
    tag = f"tables {kv_of.tolist()}"
    say(tag)
    out = _check(dw, tag)
    monkeypatch.setenv("MLKV_WORKGROUPS", "512")
    layers = _step(dw)
    # Both are within the oracle's bound; each weight is rounded to bf16
    # (2^-8 relative) against references that may differ.
    assert np.max(np.abs(out - layers)) <= 2.0 ** -7 * max(1.0, np.abs(layers).max())


def test_small_workspace_and_bf16_and_rotation():
    """A workspace that holds the layer-by-layer step's needs but not every
    run of the one-launch plan is accepted and gives fewer runs; bf16 outputs
    are the rounded fp32 ones; the rotated step leaves rotated keys."""
    dw = _prepare(12, 12, 4, 1, 64, 2, 2000, seed=5)
    say("one launch: workspaces, bf16, rotation")
    full = _step(dw)
    counters = 65536 * 4
    per_layer = 0
    for n in range(12):  # the documented layout of the layer-by-layer plan
        wg, parts = dw.map.plan(n, 2, dw.S, 64, dw.S)
        rows = 2 * 12 * parts
        up = lambda x: -(-x // 256) * 256  # noqa: E731
        per_layer = max(per_layer, counters + up(8) + up(wg * 32) + up(rows * 64 * 4) + rows * 8)
    tight = dw.ws[:per_layer].clone().zero_()
    out = _step(dw, ws=tight)
    k_gpu, v_gpu = dw.read_cache()
    k, v = dw.host["k_cache"].copy(), dw.host["v_cache"].copy()
    ref = oracle.decode_step(dw.host["q"], k, v, dw.host["k_new"], dw.host["v_new"], dw.kv_of,
                             dw.owner_of, dw.host["ctx"])
    assert np.array_equal(k_gpu, k) and np.array_equal(v_gpu, v)
    bound = step_rounding_bound(dw.host["q"], k, v, dw.kv_of, dw.host["ctx"], ref)
    check_close(out, ref, "tight workspace", bound=bound)
    check_close(full, ref, "full workspace", bound=bound)
    with pytest.raises(mlkv.MLKVError):
        _step(dw, ws=dw.ws[:counters // 2].clone())
    half = _step(dw, out_dtype=torch.bfloat16)
    assert np.array_equal(synth.f32_to_bf16(half), synth.f32_to_bf16(full))
    ws = mlkv.workspace(dw.map, 2, dw.S, 64, rotary_dims=16)
    _step(dw, ws=ws, rd=16)
    k_gpu, _ = dw.read_cache()
    k = dw.host["k_cache"].copy()
    oracle.decode_step_rope(dw.host["q"], k, v, dw.host["k_new"], dw.host["v_new"], dw.kv_of,
                            dw.owner_of, dw.host["ctx"], 16, 10000.0)
    assert np.array_equal(k_gpu, k)


@pytest.mark.parametrize("l,h,m,g,D,B,top,rd", [
    (4, 9, 2, 1, 64, 9, 900, 32),     # two blocks of rows, split runs
    (6, 12, 2, 1, 64, 130, 95, 64),   # four waves: more row chunks to turn than threads
    (12, 12, 1, 1, 64, 2, 2047, 16),  # rows in several chunks, eight runs per unit
    (8, 8, 1, 2, 128, 3, 1500, 128),  # head dim 128, every channel turned
    (12, 12, 12, 12, 64, 86, 30, 16),  # 12384 units: the angles from a table
])
def test_rotated_step_matches_oracle(l, h, m, g, D, B, top, rd):
    tag = f"one launch rotated l{l} h{h} m{m} g{g} D{D} B{B} top{top} rd{rd}"
    say(tag)
    dw = _prepare(l, h, m, g, D, B, top, seed=71 + l + h + rd)
    ws = mlkv.workspace(dw.map, B, dw.S, D, rotary_dims=rd)
    out = _step(dw, ws=ws, rd=rd)
    assert np.array_equal(out, _step(dw, ws=ws, rd=rd)), f"{tag}: a repeated step differs"
    k_gpu, v_gpu = dw.read_cache()
    k, v = dw.host["k_cache"].copy(), dw.host["v_cache"].copy()
    ref, q_rot, _ = oracle.decode_step_rope(dw.host["q"], k, v, dw.host["k_new"],
                                            dw.host["v_new"], dw.kv_of, dw.owner_of,
                                            dw.host["ctx"], rd, 10000.0, return_rotated=True)
    assert np.array_equal(k_gpu, k) and np.array_equal(v_gpu, v), f"{tag}: cache differs"
    check_close(out, ref, tag, bound=step_rounding_bound(q_rot, k, v, dw.kv_of, dw.host["ctx"],
                                                         ref))


@pytest.mark.parametrize("l,h,m,g,D,B,top", [
    (4, 8, 2, 1, 64, 9, 700),     # split runs
    (8, 8, 1, 2, 128, 9, 600),    # ... of two chunks, head dim 128
    (6, 12, 2, 1, 64, 130, 700),  # whole units on four waves
])
def test_rows_without_a_score_are_nan_and_empty_rows_zero(l, h, m, g, D, B, top):
    """A NaN query, a NaN newest key that is the only one attended, and a run
    of NaN keys make their rows NaN, as the definition does; a row that attends
    nothing is zero even then, and every other row is untouched."""
    tag = f"step without a score l{l} h{h} m{m} g{g} D{D} B{B}"
    say(tag)
    dw = _prepare(l, h, m, g, D, B, top, seed=97 + h)
    ctx, last = dw.host["ctx"], m * g - 1
    assert ctx[0] == -1 and ctx[1] == 0 and ctx[8] == top
    q, k_new, k_cache = dw.host["q"], dw.host["k_new"], dw.host["k_cache"]
    q[0, 0, 1, 3] = q[1, 7, 2, 5] = synth.BF16_NAN  # an empty sequence's, one of 65 positions
    k_new[1, 0, 9] = synth.BF16_NAN                 # the only position of sequence 1
    k_cache[last, 8, :352] = synth.BF16_NAN         # the first half of sequence 8
    dw.q, dw.k_new = mlkv.bf16_tensor(q, "cuda"), mlkv.bf16_tensor(k_new, "cuda")
    dw.cache.load_rows(k_cache, dw.host["v_cache"])
    out = _step(dw)
    k, v = k_cache.copy(), dw.host["v_cache"].copy()
    ref = oracle.decode_step(q, k, v, k_new, dw.host["v_new"], dw.kv_of, dw.owner_of, ctx)
    rows = np.isnan(ref).any(axis=-1)
    assert rows[1, 7, 2] and rows[:, 1].any() and rows[:, 8].any() and not rows[:, 0].any()
    assert np.all(np.isnan(out[rows])), f"{tag}: {np.isfinite(out[rows]).sum()} finite values"
    assert np.all(out[:, 0] == 0)
    for arr in (q, k, v):  # the rows left read none of the NaN
        arr[arr == synth.BF16_NAN] = 0
    ref[rows] = 0
    out[rows] = 0
    bound = step_rounding_bound(q, k, v, dw.kv_of, ctx, ref)
    check_close(out, ref, tag, bound=bound)


@pytest.mark.parametrize("l,h,m,g,D,B", [
    (2, 2, 2, 2, 64, 193),   # 772 units: one block of rows
    (4, 32, 1, 4, 64, 193),  # ... two blocks
    (2, 2, 2, 2, 128, 193),
    (4, 32, 1, 4, 128, 193),
])
def test_eight_waves_on_whole_units(l, h, m, g, D, B):
    """Several rounds of workgroups over sequences bounded by 64 tiles: eight
    waves a unit, here with lengths from none to a few tiles and three long."""
    tag = f"eight waves l{l} h{h} m{m} g{g} D{D}"
    say(tag)
    dw = _prepare(l, h, m, g, D, B, 60, seed=41 + D)
    long = synth.step_inputs(synth.Workload("long", l=l, h=h, m=m, g=g, D=D, B=3, ctx=2047, seed=43))
    ctx = _lengths(B, 60)
    ctx[[20, 21, 22]] = (2047, 1024, 900)
    for name in ("k_cache", "v_cache"):
        wide = np.full((m * g, B, 2048, D), synth.BF16_NAN, np.uint16)
        wide[:, :, :60] = dw.host[name][:, :, :60]
        for i, b in enumerate((20, 21, 22)):
            wide[:, b, :ctx[b]] = long[name][:, i, :ctx[b]]
        dw.host[name] = wide
    dw.host["ctx"], dw.ctx, dw.S = ctx, torch.from_numpy(ctx).cuda(), 2048
    dw.cache = mlkv.Cache.empty(m * g, B, 2048, D)
    dw.cache.load_rows(dw.host["k_cache"], dw.host["v_cache"])
    dw.ws = mlkv.workspace(dw.map, B, 2048, D)
    dw.hint = 2048
    _check(dw, tag)
