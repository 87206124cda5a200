"""GPU parity: every C-ABI compute call against the CPU oracle on the same seeded bf16 bits.

Tolerances (written here, derived in the design notes): attention max-abs 2e-2 / mean-abs 2e-3;
column sums relative 1e-3; kept-index sets exact outside a 1e-5 band around the h-th score;
compacted K/V bit-exact given the indices.
"""
import math

import ctypes
import threading

import numpy as np
import pytest
import torch

import paper_2510_25600_amd as pk
from oracle import purekv_oracle as orc
from workloads import WORKLOADS, generate, small_variant

from gpu_util import (IMPORTANCE_REL, SCORE_BAND, bits_of, check_attention, check_kept_sets, f64_of, to_dev)

pytestmark = pytest.mark.gpu

F64 = orc.bf16_bits_to_f64

SMALL = {
    "tiny_4f": WORKLOADS["tiny_4f"],
    # ragged everywhere: P = 35 (no tile alignment), N = 124 < one query tile, d = 64
    "ragged_3f": small_variant("ragged_3f"),
    # query tiles straddle frame boundaries (P = 576 = 4.5 tiles), GQA 4:1, d = 128, one ragged tail tile
    "straddle_3f": small_variant("straddle_3f", n_frames=3, patch_h=24, patch_w=24, n_text=70, n_q_heads=4,
                                 n_kv_heads=1, head_dim=128),
    # no text at all, single KV head per query head
    "notext_5f": small_variant("notext_5f", n_frames=5, patch_h=8, patch_w=8, n_text=0, n_q_heads=2, n_kv_heads=2,
                               head_dim=128),
    # long text tail so that the text rows' key lists are split across work items and merged
    "longtext_2f": small_variant("longtext_2f", n_frames=2, patch_h=16, patch_w=16, n_text=2100, n_q_heads=2,
                                 n_kv_heads=1, head_dim=128),
    # workgroup shapes of the planner: 7 stacked heads x 1 row block (one wavefront idle), split text rows
    "heads7_3f": small_variant("heads7_3f", n_frames=3, patch_h=10, patch_w=10, n_text=900, n_q_heads=7,
                               n_kv_heads=1, head_dim=128),
    # 3 stacked heads x 2 row blocks (six wavefronts), two KV heads, P = 99 straddles row blocks and key halves
    "heads3_4f": small_variant("heads3_4f", n_frames=4, patch_h=9, patch_w=11, n_text=45, n_q_heads=6,
                               n_kv_heads=2, head_dim=64),
    # 12 query heads per KV head: two groups of 6 stacked heads
    "heads12_2f": small_variant("heads12_2f", n_frames=2, patch_h=12, patch_w=12, n_text=33, n_q_heads=12,
                                n_kv_heads=1, head_dim=128),
    # More units than workgroups, so that queues hold several units and every unit switch (output of the finished
    # unit, query prefetch, state reset) is compared exhaustively, not on sampled rows as in the full-size tests:
    # 7 stacked heads x 1 row block, P = 272 straddles key tiles (91 query tiles x 6 head groups: up to three units a queue)
    "manyunits_g7": small_variant("manyunits_g7", n_frames=10, patch_h=16, patch_w=17, n_text=190, n_q_heads=42,
                                  n_kv_heads=6, head_dim=128),
    # 2 stacked heads x 4 row blocks (18 query tiles x 16 head groups), d = 64
    "manyunits_g2": small_variant("manyunits_g2", n_frames=7, patch_h=15, patch_w=20, n_text=120, n_q_heads=32,
                                  n_kv_heads=16, head_dim=64),
    # one head x 8 row blocks (5 query tiles x 64 heads), d = 64
    "manyunits_g1": small_variant("manyunits_g1", n_frames=4, patch_h=16, patch_w=16, n_text=100, n_q_heads=64,
                                  n_kv_heads=64, head_dim=64),
    # degenerate shapes: a single frame (first frame = own frame, no previous one), one patch per frame (every
    # video key is its frame's only key), a single token, and a lone video token in front of a text
    "oneframe_1f": small_variant("oneframe_1f", n_frames=1, patch_h=6, patch_w=6, n_text=10, n_q_heads=4,
                                 n_kv_heads=2, head_dim=128),
    "onepatch_9f": small_variant("onepatch_9f", n_frames=9, patch_h=1, patch_w=1, n_text=3, n_q_heads=2,
                                 n_kv_heads=1, head_dim=64),
    "single_token": small_variant("single_token", n_frames=1, patch_h=1, patch_w=1, n_text=0, n_q_heads=3,
                                  n_kv_heads=3, head_dim=128),
    "mostly_text": small_variant("mostly_text", n_frames=1, patch_h=1, patch_w=1, n_text=200, n_q_heads=8,
                                 n_kv_heads=1, head_dim=64),
}


def _plan(wl, pattern):
    return pk.Plan.for_workload(wl, pattern)


@pytest.mark.parametrize("pattern", [0, 1, 2, 3])
@pytest.mark.parametrize("name", list(SMALL))
def test_prefill_matches_oracle(name, pattern):
    wl = SMALL[name]
    inp = generate(wl, seed=11)
    print(f"[case] prefill {name} pattern={pattern} N={wl.n_tokens}", flush=True)
    plan = _plan(wl, pattern)
    out, lse = pk.purekv_st_spattn_prefill(plan, to_dev(inp.q), to_dev(inp.k), to_dev(inp.v), want_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = orc.masked_attention(F64(inp.q), F64(inp.k), F64(inp.v), wl.n_frames, wl.patches, wl.n_text,
                                        pattern)
    check_attention(f64_of(out), ref, f"{name}/p{pattern}")
    assert np.abs(f64_of(lse) - ref_lse).max() < 2e-3
    if name == "longtext_2f":
        assert plan.counts()["n_split_qtiles"] > 0  # the merge path ran
    if name.startswith("manyunits"):
        c = plan.counts()
        assert max(len(plan.queue(g)) for g in range(c["n_workgroups"])) >= 2  # some queue switches units


@pytest.mark.parametrize("pattern", [0, 1, 2, 3])
@pytest.mark.parametrize("name", list(SMALL))
def test_prefill_workgroup_shapes(name, pattern):
    """A shape with few units is planned with fewer wavefronts per workgroup, as far as every unit still has a compute unit.  The
    same heads repeated until that ends: every shape on the way, the full one among them, against the oracle of the heads
    themselves."""
    wl = SMALL[name]
    inp = generate(wl, seed=11)
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    ref, ref_lse = orc.masked_attention(F64(inp.q), F64(inp.k), F64(inp.v), wl.n_frames, wl.patches, wl.n_text, pattern)
    seen, times = set(), 1
    while True:
        hq, hkv = wl.n_q_heads * times, wl.n_kv_heads * times
        plan = pk.Plan(wl.n_frames, wl.patch_h, wl.patch_w, wl.n_text, hq, hkv, wl.head_dim, pattern)
        c = plan.counts()
        shape = (c["stacked_heads"], c["row_blocks"])
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
        lists = c["n_qtiles"] * c["n_head_groups"]
        if shape not in seen:
            print(f"[case] prefill {name} pattern={pattern} x{times} shape={shape}", flush=True)
            assert shape[0] * shape[1] > 4 or lists <= n_cu
            out, lse = pk.purekv_st_spattn_prefill(plan, *(x.repeat(times, 1, 1) for x in (q, k, v)), want_lse=True)
            torch.cuda.synchronize()
            for part in (0, times // 2, times - 1):
                rows = slice(part * wl.n_q_heads, (part + 1) * wl.n_q_heads)
                check_attention(f64_of(out[rows]), ref, f"{name}/p{pattern} x{times}")
                assert np.abs(f64_of(lse[rows]) - ref_lse).max() < 2e-3
        seen.add(shape)
        plan.close()
        if lists > 2 * n_cu:
            break
        times *= 2
    assert any(a * b > 4 for a, b in seen)


@pytest.mark.parametrize("want_lse", [False, True])
@pytest.mark.parametrize("dim", [64, 128])
@pytest.mark.parametrize("frames,patch_h,patch_w,text", [(2, 5, 5, 0), (2, 7, 7, 2), (3, 7, 8, 12)])
def test_prefill_units_of_one_to_three_steps(frames, patch_h, patch_w, text, dim, want_lse):
    """Workgroups that run two or three units of one, two or three key tiles each: every step of such a queue begins or ends
    a unit or requests the next one's query rows, and the pipeline never reaches its plain middle."""
    wl = small_variant("short_units", n_frames=frames, patch_h=patch_h, patch_w=patch_w, n_text=text, n_q_heads=700,
                       n_kv_heads=700, head_dim=dim)
    inp = generate(wl, seed=5)
    for pattern in (pk.PATTERN_DENSE, pk.PATTERN_ST):
        plan = _plan(wl, pattern)
        assert plan.counts()["n_workgroups"] < 700
        got = pk.purekv_st_spattn_prefill(plan, to_dev(inp.q), to_dev(inp.k), to_dev(inp.v), want_lse=want_lse)
        torch.cuda.synchronize()
        ref, ref_lse = orc.masked_attention(F64(inp.q), F64(inp.k), F64(inp.v), wl.n_frames, wl.patches, wl.n_text, pattern)
        check_attention(f64_of(got[0] if want_lse else got), ref, f"short units {wl.n_tokens}/d{dim}/p{pattern}")
        if want_lse:
            assert np.abs(f64_of(got[1]) - ref_lse).max() < 2e-3


@pytest.mark.parametrize("pattern", [0, 3])
@pytest.mark.parametrize("name,w", [("manyunits_g7", 190), ("manyunits_g7", 37), ("manyunits_g2", 120), ("manyunits_g2", 1),
                                    ("manyunits_g1", 100), ("manyunits_g1", 300), ("tiny_4f", 32), ("longtext_2f", 64)])
def test_window_plan_prefill_and_importance(name, w, pattern):
    """A window plan: outputs as for any plan; the log-sum-exp of the last w rows only, every other element of the
    buffer untouched; the importance read from it.  The larger shapes have more units than workgroups, so their
    plans are divided and the kernel with both copies of the tile loop runs."""
    wl = SMALL[name]
    inp = generate(wl, seed=21)
    n = wl.n_tokens
    print(f"[case] window plan {name} pattern={pattern} w={w} N={n}", flush=True)
    plan = pk.Plan.for_workload(wl, pattern, lse_window=w)
    c = plan.counts()
    # these are the cases meant to exercise the divided kernel, at both head dimensions (the planner leaves a plan whole
    # when the window's tiles are more than a quarter of the work, or when there are fewer units than workgroups)
    if (name, w, pattern) in {("manyunits_g7", 37, 0), ("manyunits_g7", 37, 3), ("manyunits_g2", 120, 0),
                              ("manyunits_g2", 1, 0), ("manyunits_g2", 1, 3)}:
        assert c["lse_queue0"] > 0, "this case is meant to exercise the divided kernel"
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    sentinel = -12345.0
    lse = torch.full((wl.n_q_heads, n), sentinel, dtype=torch.float32, device="cuda")
    out, _ = pk.purekv_st_spattn_prefill(plan, q, k, v, lse=lse)
    torch.cuda.synchronize()
    qf, kf, vf = F64(inp.q), F64(inp.k), F64(inp.v)
    ref, ref_lse = orc.masked_attention(qf, kf, vf, wl.n_frames, wl.patches, wl.n_text, pattern)
    check_attention(f64_of(out), ref, f"window {name}/p{pattern}/w{w}")
    got_lse = f64_of(lse)
    assert np.all(got_lse[:, :n - w] == sentinel), "rows before the window were written"
    assert np.abs(got_lse[:, n - w:] - ref_lse[:, n - w:]).max() < 2e-3
    # the same call without the log-sum-exp, and again with it: same output bits (the division changes who runs what,
    # never what is computed for a row)
    out2 = pk.purekv_st_spattn_prefill(plan, q, k, v)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(out), bits_of(out2))
    cs = pk.purekv_lowlayer_importance(plan, q, k, lse, w)
    torch.cuda.synchronize()
    ref_c = orc.window_column_sums(qf, kf, wl.n_frames, wl.patches, wl.n_text, pattern, w)
    got_c = f64_of(cs)
    if ref_c.size:
        assert np.all(np.abs(got_c - ref_c) <= IMPORTANCE_REL * np.maximum(np.abs(ref_c), 1e-12))
    # a window wider than the plan's is refused: those rows of lse were never written
    if w < n:
        with pytest.raises(pk.PureKVError) as e:
            pk.purekv_lowlayer_importance(plan, q, k, lse, w + 1)
        assert e.value.status == pk.EINVAL
    # the V norms asked for together with the window's log-sum-exp come from their own pass: same values
    vn = torch.zeros((wl.n_kv_heads, n), dtype=torch.float32, device="cuda")
    lse3 = torch.full_like(lse, sentinel)
    out3, _ = pk.purekv_st_spattn_prefill(plan, q, k, v, lse=lse3, vnorm2=vn)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(out), bits_of(out3)) and torch.equal(lse, lse3)
    ref_vn = (vf * vf).sum(-1)
    assert np.abs(f64_of(vn) - ref_vn).max() <= 2e-6 * max(1.0, ref_vn.max())


def test_prefill_is_deterministic_and_output_buffer_reuse():
    wl = SMALL["straddle_3f"]
    inp = generate(wl, seed=3)
    plan = _plan(wl, 3)
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    a = pk.purekv_st_spattn_prefill(plan, q, k, v)
    b = torch.full_like(a, float("nan"))
    pk.purekv_st_spattn_prefill(plan, q, k, v, out=b)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(a), bits_of(b))


@pytest.mark.parametrize("d,pattern,window", [(128, 0, 0), (128, 3, 0), (64, 0, 0), (64, 3, 0), (128, 0, 40), (64, 0, 40)])
def test_prefill_takes_a_large_key_as_reference(d, pattern, window):
    """Every score is 0 but one key's, beyond the first tile, which is log2(16 / 15 * 2^9) = 9.09 in log2 units: more than the 8
    by which a key may exceed a row's softmax reference, so it becomes the reference and its own probability is 1.  The
    other probabilities are then 15 / 16 * 2^-9.  bf16 holds both exactly, so the weights carry no rounding of the
    probabilities; against a reference that stays a whole number of units from the first tile's maximum, 16 / 15 is 3.4e-3
    off and a row's two halves, +1 and -1, cancel to less than that."""
    from workloads import f32_to_bf16_bits
    f, ph, pw, t, hq, hkv, dom = 3, 15, 21, 900, 2, 1, 150
    n = f * ph * pw + t
    q, k, v = (np.zeros((x, n, d), dtype=np.float32) for x in (hq, hkv, hkv))
    x, parts = math.log2(16.0 / 15.0 * 512.0), []
    for _ in range(3):   # as a sum of three bf16 numbers
        parts.append(float(F64(f32_to_bf16_bits(np.array([x], dtype=np.float32)))[0]))
        x -= parts[-1]
    q[:, :, :3] = 1.0
    k[:, dom, :3] = parts
    v[:] = -1.0
    v[:, dom] = 1.0
    q, k, v = f32_to_bf16_bits(q), f32_to_bf16_bits(k), f32_to_bf16_bits(v)
    plan = pk.Plan(f, ph, pw, t, hq, hkv, d, pattern, math.log(2.0), lse_window=window)
    lse = torch.zeros((hq, n), dtype=torch.float32, device="cuda")
    out, _ = pk.purekv_st_spattn_prefill(plan, to_dev(q), to_dev(k), to_dev(v), lse=lse)
    torch.cuda.synchronize()
    ref, _ = orc.masked_attention(F64(q), F64(k), F64(v), f, ph * pw, t, pattern, scale=math.log(2.0))
    assert (np.abs(ref[:, dom:]) < 0.2).any()
    # the output's own rounding (half a unit of 8 significant bits), and fp32 sums of a thousand terms beside it
    over = np.abs(f64_of(out) - ref) - (2.0 ** -8 * np.abs(ref) + 5e-5)
    assert over.max() <= 0.0, f"error {over.max():.3g} over the bound in {(over > 0.0).sum()} elements"


@pytest.mark.parametrize("d,step", [(128, 0.75), (128, 12.0), (64, 12.0), (64, -0.75), (128, 300.0)])
@pytest.mark.parametrize("pattern", [0, 3])
def test_prefill_reference_is_raised(pattern, d, step):
    """Scores that grow (or fall) by `step` log2 units every 16 keys: the softmax reference has to be raised never, every few
    tiles, or by more than a float's exponent range at once (300: probabilities against the reference before would
    overflow), also in the slices of split lists."""
    from workloads import f32_to_bf16_bits
    rng = np.random.default_rng(int(d + 8 * abs(step)))
    f, ph, pw, t, hq, hkv = 3, 9, 11, 470, 2, 1
    n = f * ph * pw + t
    q, k, v = (rng.standard_normal((x, n, d)).astype(np.float32) for x in (hq, hkv, hkv))
    # two columns carry the trend (a coarse and a fine part, so that bf16 keeps it): q = 1 there
    trend = np.round(step * np.arange(n) // 16 * math.log(2.0) * math.sqrt(d) * 16.0) / 16.0
    hi = np.round(trend / 64.0) * 64.0
    q[:, :, 0] = q[:, :, 1] = 1.0
    k[:, :, 0], k[:, :, 1] = hi, trend - hi
    q, k, v = f32_to_bf16_bits(q), f32_to_bf16_bits(k), f32_to_bf16_bits(v)
    plan = pk.Plan(f, ph, pw, t, hq, hkv, d, pattern)
    out, lse = pk.purekv_st_spattn_prefill(plan, to_dev(q), to_dev(k), to_dev(v), want_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = orc.masked_attention(F64(q), F64(k), F64(v), f, ph * pw, t, pattern)
    check_attention(f64_of(out), ref, f"trend {step} d={d} p{pattern}")
    # the fp32 sum of a dot product of magnitude |s| is off by a few 2^-24 |s|
    assert (np.abs(f64_of(lse) - ref_lse) <= 2e-3 + 2.0 ** -21 * np.abs(ref_lse)).all()


@pytest.mark.parametrize("pattern", [0, 3])
@pytest.mark.parametrize("frames,patch_h,patch_w,text,dim", [(4, 9, 11, 700, 128), (2, 16, 16, 600, 64)])
def test_prefill_rows_whose_scores_are_all_minus_infinity(frames, patch_h, patch_w, text, dim, pattern):
    """A row none of whose scores is finite has no weights: its output is 0 and its log-sum-exp -inf, whether its key list
    is run whole or in slices; and a slice without a finite score adds nothing to the others."""
    from workloads import f32_to_bf16_bits
    wl = small_variant("minus_inf", n_frames=frames, patch_h=patch_h, patch_w=patch_w, n_text=text, n_q_heads=4, n_kv_heads=2,
                       head_dim=dim)
    n, half = wl.n_tokens, wl.n_tokens // 2
    rng = np.random.default_rng(dim)
    q, k, v = (rng.standard_normal((h, n, dim)).astype(np.float32) for h in (4, 2, 2))
    q[:, :, 0] = 1.0
    k[:, :, 0] = 0.0
    k[0, :, 0], k[1, :half, 0] = -np.inf, -np.inf     # no key of KV head 0 has a finite score, no key before `half` of 1
    qb, kb, vb = (f32_to_bf16_bits(x) for x in (q, k, v))
    plan = _plan(wl, pattern)
    assert plan.counts()["n_split_qtiles"] > 0 and any(plan.item(i)[4] == 1 for i in range(plan.counts()["n_items"]))
    out, lse = pk.purekv_st_spattn_prefill(plan, to_dev(qb), to_dev(kb), to_dev(vb), want_lse=True)
    torch.cuda.synchronize()
    out, lse = f64_of(out), f64_of(lse)
    mask = orc.st_mask(frames, patch_h * patch_w, text, pattern)
    dead = ~mask[:, half:].any(axis=1)                # rows of the second KV head's query heads without a finite score
    assert dead.any() and not dead.all()
    assert not out[:2].any() and np.isneginf(lse[:2]).all()
    assert not out[2:, dead].any() and np.isneginf(lse[2:, dead]).all()
    kf = F64(kb)
    kf[:, :, 0] = np.where(np.isneginf(kf[:, :, 0]), -1e9, 0.0)
    ref, ref_lse = orc.masked_attention(F64(qb), kf, F64(vb), frames, patch_h * patch_w, text, pattern)
    check_attention(out[2:, ~dead], ref[2:, ~dead], f"-inf scores d={dim} p={pattern}")
    assert np.abs(lse[2:, ~dead] - ref_lse[2:, ~dead]).max() < 2e-3


def test_prefill_custom_scale():
    wl = SMALL["ragged_3f"]
    inp = generate(wl, seed=5)
    plan = pk.Plan(wl.n_frames, wl.patch_h, wl.patch_w, wl.n_text, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, 3, 0.05)
    out = pk.purekv_st_spattn_prefill(plan, to_dev(inp.q), to_dev(inp.k), to_dev(inp.v))
    ref, _ = orc.masked_attention(F64(inp.q), F64(inp.k), F64(inp.v), wl.n_frames, wl.patches, wl.n_text, 3,
                                  scale=float(np.float32(0.05)))
    check_attention(f64_of(out), ref, "custom scale")


@pytest.mark.parametrize("name,pattern,w", [
    ("tiny_4f", 0, 32), ("tiny_4f", 3, 32), ("tiny_4f", 3, 100), ("tiny_4f", 2, 200), ("tiny_4f", 0, 288),
    ("ragged_3f", 3, 19), ("ragged_3f", 1, 50), ("straddle_3f", 3, 70), ("straddle_3f", 0, 700),
    ("notext_5f", 3, 33), ("longtext_2f", 0, 2100),
    ("oneframe_1f", 3, 10), ("oneframe_1f", 3, 30), ("oneframe_1f", 2, 46), ("onepatch_9f", 3, 5), ("onepatch_9f", 1, 12),
    ("single_token", 3, 1), ("mostly_text", 3, 64), ("mostly_text", 3, 201), ("heads7_3f", 3, 900), ("heads3_4f", 2, 150),
])
def test_importance_matches_oracle(name, pattern, w):
    wl = SMALL[name]
    inp = generate(wl, seed=12)
    print(f"[case] importance {name} pattern={pattern} w={w}", flush=True)
    plan = _plan(wl, pattern)
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    _, lse = pk.purekv_st_spattn_prefill(plan, q, k, v, want_lse=True)
    c = pk.purekv_lowlayer_importance(plan, q, k, lse, w)
    torch.cuda.synchronize()
    ref = orc.window_column_sums(F64(inp.q), F64(inp.k), wl.n_frames, wl.patches, wl.n_text, pattern, w)
    got = f64_of(c)
    assert got.shape == ref.shape
    if ref.size:
        assert np.all(np.abs(got - ref) <= IMPORTANCE_REL * np.maximum(np.abs(ref), 1e-12)), \
            f"worst rel {np.max(np.abs(got - ref) / np.maximum(np.abs(ref), 1e-12)):.3g}"
    # masked-out pairs contribute exactly nothing: a column no window row can see is exactly 0
    assert np.all(got[ref == 0] == 0)


@pytest.mark.parametrize("nv,w,hq,hkv", [(4100, 40, 8, 8), (2817, 31, 12, 12), (5569, 97, 12, 6), (3300, 40, 40, 40)])
def test_importance_wide_workgroups(nv, w, hq, hkv):
    """Key counts whose 128-key tiles are a few more than the chip has compute units (264, 276, 264): 192 keys per workgroup
    then, here with ragged last tiles and odd and even numbers of query blocks; 1040 tiles: three rounds of 192 keys."""
    rng = np.random.default_rng(nv + w)
    n = nv + w
    from workloads import f32_to_bf16_bits
    q, k, v = (f32_to_bf16_bits(rng.standard_normal((x, n, 128)).astype(np.float32)) for x in (hq, hkv, hkv))
    plan = pk.Plan(1, 1, nv, w, hq, hkv, 128, 0)
    dq, dk = to_dev(q), to_dev(k)
    _, lse = pk.purekv_st_spattn_prefill(plan, dq, dk, to_dev(v), want_lse=True)
    c = pk.purekv_lowlayer_importance(plan, dq, dk, lse, w)
    ref = orc.window_column_sums(F64(q), F64(k), 1, nv, w, 0, w)
    assert np.all(np.abs(f64_of(c) - ref) <= IMPORTANCE_REL * ref)


@pytest.mark.parametrize("n_keys,h", [(256, 25), (256, 0), (256, 256), (1000, 1), (5000, 999), (40000, 8000)])
def test_topk_exact_on_given_scores(n_keys, h):
    """Stage-isolated: identical fp32 scores on both sides, so the kept sets must be identical (ties included)."""
    w = 16
    n = n_keys + w
    plan = pk.Plan(1, 1, n_keys, w, 3, 3, 64, 0)  # geometry only carries N and Hkv here
    rng = np.random.default_rng(n_keys + h)
    s = rng.random((3, n_keys)).astype(np.float32)
    s[1] = np.round(s[1] * 8) / 8                 # heavy ties
    s[2, ::3] = 0.0                               # zeros, some negative zero
    s[2, 3::6] = -0.0
    idx = pk.purekv_topk_select(plan, torch.from_numpy(s).cuda(), None, w, h)
    torch.cuda.synchronize()
    ref = orc.topk_select(s.astype(np.float64), h, n, w)
    assert np.array_equal(idx.cpu().numpy(), ref)


@pytest.mark.parametrize("n_keys", [8192, 8193, 16384, 20000, 32768, 32769, 50001])
def test_topk_row_lengths_across_kernel_variants(n_keys):
    """Row lengths on both sides of every switch between the register-resident variants (8, 16, 32 scores per
    thread) and the streaming variant of the selection kernel; heavy ties in one head."""
    w = 8
    plan = pk.Plan(1, 1, n_keys, w, 2, 2, 64, 0)
    rng = np.random.default_rng(n_keys)
    s = rng.random((2, n_keys)).astype(np.float32)
    s[1] = np.round(s[1] * 16) / 16
    for h in (1, n_keys // 5, n_keys):
        idx = pk.purekv_topk_select(plan, torch.from_numpy(s).cuda(), None, w, h)
        ref = orc.topk_select(s.astype(np.float64), h, n_keys + w, w)
        assert np.array_equal(idx.cpu().numpy(), ref), (n_keys, h)


@pytest.mark.parametrize("n_keys", [1, 63, 1025, 8191, 30001])
@pytest.mark.parametrize("crowd", [1, 2, 31, 32, 33, 64])
def test_topk_crowd_at_the_threshold(n_keys, crowd):
    """`crowd` keys that differ from each other in their last bits only (some of them equal), the h-th largest among them, in
    rows that end inside a block of 1024: the radix passes end in a list of at most 32 candidates or in one pass more.
    For each row, the h that ends just above its crowd, at the crowd's first, middle and last key, and just below."""
    if crowd > n_keys:
        pytest.skip("row shorter than the crowd")
    w = 8
    plan = pk.Plan(1, 1, n_keys, w, 3, 3, 64, 0)
    rng = np.random.default_rng(1000 * n_keys + crowd)
    s = rng.standard_normal((3, n_keys)).astype(np.float32)
    s[1] = np.exp(s[1])
    bits = s.view(np.int32)
    at = rng.permutation(n_keys)[:crowd]
    base = np.float32(0.75).view(np.int32)
    bits[0, at] = base + rng.integers(0, 256, crowd)     # distinct ones and ties
    bits[1, at] = base + np.arange(crowd)                # all distinct
    bits[2, at] = base + (np.arange(crowd) % 3 == 0)     # two values
    for k in range(3):
        above = int((s[k] > s[k, at].max()).sum())
        in_crowd = {above + 1, above + (crowd + 1) // 2, above + crowd}
        ranked = np.sort(s[k])[::-1]
        for h in sorted({1, n_keys, above, above + crowd + 1} | in_crowd):
            if not 1 <= h <= n_keys:
                continue
            assert h not in in_crowd or s[k, at].min() <= ranked[h - 1] <= s[k, at].max()
            idx = pk.purekv_topk_select(plan, torch.from_numpy(s).cuda(), None, w, h)
            ref = orc.topk_select(s.astype(np.float64), h, n_keys + w, w)
            assert np.array_equal(idx.cpu().numpy(), ref), (k, h)


def test_topk_negative_and_mixed_scores():
    w, n_keys = 8, 3000
    plan = pk.Plan(1, 1, n_keys, w, 2, 2, 64, 0)
    rng = np.random.default_rng(9)
    s = rng.standard_normal((2, n_keys)).astype(np.float32)
    s[1] = -np.abs(s[1])
    for h in (1, 500, 2999):
        idx = pk.purekv_topk_select(plan, torch.from_numpy(s).cuda(), None, w, h)
        ref = orc.topk_select(s.astype(np.float64), h, n_keys + w, w)
        assert np.array_equal(idx.cpu().numpy(), ref)


@pytest.mark.parametrize("d,n_keys", [(64, 1), (64, 127), (64, 1023), (64, 1024), (64, 1025), (128, 63), (128, 511), (128, 512), (128, 513)])
@pytest.mark.parametrize("layers", [1, 3])
def test_selection_that_forms_its_scores(d, n_keys, layers):
    """Up to 128 KB of V rows per KV head the selecting workgroup forms the scores itself: bit for bit those of the score
    kernel (the same rows at the head of a longer layer), and the choice that follows from them."""
    w, longer, hkv = 9, 1200, 3
    rng = np.random.default_rng(n_keys + d + layers)
    v = torch.from_numpy(rng.standard_normal((layers, hkv, n_keys + longer + w, d)).astype(np.float32)).bfloat16().cuda()
    c = torch.from_numpy(np.exp(rng.standard_normal((hkv, n_keys + longer))).astype(np.float32)).cuda()
    small, large = pk.Plan(1, 1, n_keys, w, hkv, hkv, d, 0), pk.Plan(1, 1, n_keys + longer, w, hkv, hkv, d, 0)
    _, s_ref = pk.purekv_topk_select(large, c, v, w, 1, want_scores=True)
    s_ref = s_ref.reshape(layers, hkv, -1)[:, :, :n_keys]
    vs, cs = v[:, :, :n_keys + w].contiguous(), c[:, :n_keys].contiguous()
    for h in sorted({0, 1, n_keys // 3, n_keys}):
        idx, s = pk.purekv_topk_select(small, cs, vs, w, h, want_scores=True)
        again = pk.purekv_topk_select(small, cs, vs, w, h)
        assert torch.equal(s.reshape(s_ref.shape).view(torch.int32), s_ref.contiguous().view(torch.int32))
        assert torch.equal(idx, again)
        for l in range(layers):
            ref = orc.topk_select(s_ref[l].cpu().numpy().astype(np.float64), h, n_keys + w, w)
            assert np.array_equal(idx.reshape(layers, hkv, -1)[l].cpu().numpy(), ref)


@pytest.mark.parametrize("n_keys", [65, 1024, 1025, 2049, 4097, 6144, 6145, 16385])
def test_topk_exact_on_scores_of_any_range(n_keys):
    """Rows over the whole range of fp32 (infinities and the smallest and largest numbers of both signs), within a few units in
    the last place (also but for one key), of one value (likewise), and of two values that share the threshold among them."""
    w, rng = 5, np.random.default_rng(n_keys)
    bits = rng.integers(0, 2 ** 32, n_keys, dtype=np.uint64).astype(np.uint32)
    wide = bits.view(np.float32).copy()
    wide[~np.isfinite(wide)] = np.inf
    wide[:7] = [np.inf, -np.inf, 3.4028235e38, -3.4028235e38, 1e-45, -1e-45, -0.0]
    near = (np.float32(1.5).view(np.uint32) + rng.integers(0, 40, n_keys).astype(np.uint32)).view(np.float32)
    one = np.full(n_keys, -2.5, np.float32)
    two = np.where(rng.random(n_keys) < 0.5, np.float32(0.25), np.float32(0.75)).astype(np.float32)
    but_one = one.copy()
    but_one[n_keys // 2] = 1e30
    near_but_one = near.copy()   # all but one key in one bin of the first pass
    near_but_one[n_keys // 3] = 1e30
    s = np.stack([wide, near, one, two, but_one, near_but_one])
    plan = pk.Plan(1, 1, n_keys, w, 6, 6, 64, 0)
    for h in (1, 2, 65, n_keys // 5 + 1, n_keys // 2, n_keys - 1, n_keys):
        idx = pk.purekv_topk_select(plan, torch.from_numpy(s).cuda(), None, w, min(h, n_keys))
        assert np.array_equal(idx.cpu().numpy(), orc.topk_select(s.astype(np.float64), min(h, n_keys), n_keys + w, w)), h


def _graph_us(call, calls=20):
    """Median time of a call, us, of `calls` in a row from a HIP graph (no host in between)."""
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        call()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for _ in range(calls):
            call()
    times = []
    for _ in range(9):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / calls)
    return sorted(times)[len(times) // 2]


@pytest.mark.parametrize("n_keys", [1025, 4097, 8192, 16384, 16385])
def test_selection_of_crowded_rows(n_keys):
    """Rows whose keys share a bin or two of the histogram: weights that are exactly 0 (the threshold among them, above them),
    four values, all but one within a few units in the last place, and those beside a spread.  Exact, and for the longer rows not
    much slower than rows that spread out: additions of a wavefront to one bin, one lane at a time, took four to six times as long
    (now 1.2 to 1.9)."""
    w, rng = 7, np.random.default_rng(n_keys)
    spread = np.exp(1.2 * rng.standard_normal(n_keys)).astype(np.float32)
    zeros = np.where(rng.random(n_keys) < 0.9, np.float32(0), spread)
    alike = (np.float32(1.5).view(np.uint32) + rng.integers(0, 8, n_keys).astype(np.uint32)).view(np.float32)
    alike[n_keys // 2] = 1e30
    rows = {"spread": spread, "zeros": zeros, "four values": rng.integers(1, 5, n_keys).astype(np.float32), "alike": alike,
            "alike and spread": np.where(rng.random(n_keys) < 0.4, alike, spread), "-zeros": -zeros}
    plan, one = pk.Plan(1, 1, n_keys, w, len(rows), len(rows), 64, 0), pk.Plan(1, 1, n_keys, w, 4, 4, 64, 0)
    s = np.stack(list(rows.values()))
    for h in (1, n_keys // 20, n_keys // 10, n_keys // 5, n_keys // 2, n_keys - 1):
        idx = pk.purekv_topk_select(plan, torch.from_numpy(s).cuda(), None, w, h)
        assert np.array_equal(idx.cpu().numpy(), orc.topk_select(s.astype(np.float64), h, n_keys + w, w)), h
    if n_keys < 8192:
        return
    times = {}
    for name, row in rows.items():
        c = torch.from_numpy(np.stack([row] * 4)).cuda()
        out = torch.empty((1, 4, n_keys // 5 + w), dtype=torch.int32, device="cuda")
        times[name] = _graph_us(lambda: pk.purekv_topk_select(one, c, None, w, n_keys // 5, idx_out=out))
    print(f"[case] {n_keys} keys, us: {times}", flush=True)
    assert max(times.values()) <= 2.5 * times["spread"], times


@pytest.mark.parametrize("name", ["tiny_4f", "ragged_3f", "straddle_3f"])
def test_vnorm_scores_and_selection_layers(name):
    """Eq. 3 / Eq. 4: several layers' V share one C; scores within fp32 rounding, kept sets exact outside the band."""
    wl = SMALL[name]
    n, w = wl.n_tokens, wl.window
    h = max(1, orc.budget(n, w, 0.3))
    layers = [generate(wl, seed=20 + l) for l in range(3)]
    rng = np.random.default_rng(1)
    c = rng.random((wl.n_kv_heads, n - w)).astype(np.float32)
    plan = _plan(wl, 3)
    v_all = torch.stack([to_dev(x.v) for x in layers])
    idx, s = pk.purekv_topk_select(plan, torch.from_numpy(c).cuda(), v_all, w, h, want_scores=True)
    idx2 = pk.purekv_topk_select(plan, torch.from_numpy(c).cuda(), v_all, w, h)  # workspace path
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx2.cpu().numpy())
    for l, x in enumerate(layers):
        s_ref = orc.vnorm_scores(c.astype(np.float64), F64(x.v))
        assert np.all(np.abs(f64_of(s[l]) - s_ref) <= 2e-6 * np.abs(s_ref) + 1e-30)
        check_kept_sets(idx[l].cpu().numpy(), orc.topk_select(s_ref, h, n, w), s_ref, h)


@pytest.mark.parametrize("name", ["tiny_4f", "ragged_3f", "straddle_3f"])
def test_compaction_bit_exact_and_append(name):
    wl = SMALL[name]
    n, w = wl.n_tokens, wl.window
    h = orc.budget(n, w, 0.4)
    layers = [generate(wl, seed=30 + l) for l in range(2)]
    rng = np.random.default_rng(2)
    idx = np.stack([orc.topk_select(rng.random((wl.n_kv_heads, n - w)), h, n, w) for _ in layers])
    plan = _plan(wl, 3)
    k_all = torch.stack([to_dev(x.k) for x in layers])
    v_all = torch.stack([to_dev(x.v) for x in layers])
    cap = h + w + 3
    kc = torch.zeros((2, wl.n_kv_heads, cap, wl.head_dim), dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    pk.purekv_kv_compact(plan, k_all, v_all, torch.from_numpy(idx).cuda(), cap=cap, kc=kc, vc=vc)
    torch.cuda.synchronize()
    for l, x in enumerate(layers):
        kr, vr = orc.compact(x.k, x.v, idx[l])
        assert np.array_equal(bits_of(kc[l])[:, :h + w], kr) and np.array_equal(bits_of(vc[l])[:, :h + w], vr)
        assert not bits_of(kc[l])[:, h + w:].any()  # rows beyond n_keep untouched
    # append one decoded token to layer 0's cache
    x = layers[0]
    n1 = pk.purekv_kv_append(plan, to_dev(x.k_new[0]) if x.k_new.shape[0] else to_dev(x.k[:, 0]),
                             to_dev(x.v_new[0]) if x.v_new.shape[0] else to_dev(x.v[:, 0]), kc[0], vc[0], h + w)
    torch.cuda.synchronize()
    assert n1 == h + w + 1
    src = x.k_new[0] if x.k_new.shape[0] else x.k[:, 0]
    assert np.array_equal(bits_of(kc[0])[:, h + w], src)


@pytest.mark.parametrize("hq,hkv,d,n_cached", [(2, 1, 64, 57), (28, 4, 128, 1690), (32, 8, 128, 948), (12, 1, 128, 5),
                                               (4, 4, 64, 1), (9, 3, 128, 333), (40, 2, 128, 300), (34, 2, 64, 129),
                                               (28, 4, 128, 128), (28, 4, 128, 6800), (4, 1, 64, 17000), (6, 2, 128, 33000)])
def test_decode_matches_oracle(hq, hkv, d, n_cached):
    rng = np.random.default_rng(n_cached)
    from workloads import f32_to_bf16_bits
    q = f32_to_bf16_bits(rng.standard_normal((hq, d)).astype(np.float32))
    cap = n_cached + 7
    kc = f32_to_bf16_bits(rng.standard_normal((hkv, cap, d)).astype(np.float32))
    vc = f32_to_bf16_bits(rng.standard_normal((hkv, cap, d)).astype(np.float32))
    plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
    out = pk.purekv_decode_attn(plan, to_dev(q), to_dev(kc), to_dev(vc), n_cached)
    torch.cuda.synchronize()
    ref = orc.decode_attention(F64(q), F64(kc)[:, :n_cached], F64(vc)[:, :n_cached])
    check_attention(f64_of(out), ref, "decode")


@pytest.mark.parametrize("hq,hkv,d,n0,steps", [(28, 4, 128, 1689, 3), (40, 2, 64, 126, 5), (8, 8, 128, 0, 3),
                                               (12, 3, 128, 255, 3)])
def test_decode_step_appends_and_attends(hq, hkv, d, n0, steps):
    """The fused step = append + attention: the cache must equal the one the separate append call builds, bit for
    bit, the output must match the oracle on the grown cache, and consecutive calls (the arrival counters reset
    themselves) must keep doing so, also across a 256-key chunk boundary."""
    from workloads import f32_to_bf16_bits
    rng = np.random.default_rng(1000 * hq + n0)
    bits = lambda *shape: f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))  # noqa: E731
    cap = n0 + steps + 2
    kc_h, vc_h = bits(hkv, cap, d), bits(hkv, cap, d)
    kc, vc = to_dev(kc_h), to_dev(vc_h)           # fused path
    kc2, vc2 = to_dev(kc_h), to_dev(vc_h)         # separate append + attention
    plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
    for t in range(steps):
        q, kn, vn = bits(hq, d), bits(hkv, d), bits(hkv, d)
        n = n0 + t
        out = pk.purekv_decode_step(plan, to_dev(q), to_dev(kn), to_dev(vn), kc, vc, n)
        pk.purekv_kv_append(plan, to_dev(kn), to_dev(vn), kc2, vc2, n)
        out2 = pk.purekv_decode_attn(plan, to_dev(q), kc2, vc2, n + 1)
        torch.cuda.synchronize()
        kc_h[:, n], vc_h[:, n] = kn, vn
        assert np.array_equal(bits_of(kc)[:, :n + 1], kc_h[:, :n + 1]) and np.array_equal(bits_of(kc), bits_of(kc2))
        assert np.array_equal(bits_of(vc)[:, :n + 1], vc_h[:, :n + 1]) and np.array_equal(bits_of(vc), bits_of(vc2))
        assert np.array_equal(bits_of(out), bits_of(out2))   # same kernel, same order of operations
        ref = orc.decode_attention(F64(q), F64(kc_h)[:, :n + 1], F64(vc_h)[:, :n + 1])
        check_attention(f64_of(out), ref, f"decode step {t}")


@pytest.mark.parametrize("hq,hkv,d,n0", [
    (16, 1, 128, 256 * 17),       # sixteen heads: one group of lanes per head, a second batch of partial outputs
    (2, 1, 64, 64 * 256 + 2),     # 65 chunks of 64-wide heads: a second pass of the final merge
    (7, 1, 128, 128 * 256),       # 129 chunks of 128-wide heads: likewise, the last chunk is the appended key alone
    (17, 1, 64, 256 * 3 + 31),    # a second block of heads with one head in it
])
def test_decode_step_merges_many_chunks(hq, hkv, d, n0):
    """The merge of the chunks at its edges, twice on one workspace (the counters are left at zero)."""
    from workloads import f32_to_bf16_bits
    rng = np.random.default_rng(hq + n0)
    bits = lambda *shape: f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))  # noqa: E731
    plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
    q, kn, vn = bits(hq, d), bits(hkv, d), bits(hkv, d)
    kc_h, vc_h = bits(hkv, n0 + 1, d), bits(hkv, n0 + 1, d)
    kc, vc = to_dev(kc_h), to_dev(vc_h)
    outs = [pk.purekv_decode_step(plan, to_dev(q), to_dev(kn), to_dev(vn), kc, vc, n0) for _ in range(2)]
    torch.cuda.synchronize()
    kc_h[:, n0], vc_h[:, n0] = kn, vn
    assert np.array_equal(bits_of(kc), kc_h) and np.array_equal(bits_of(vc), vc_h)
    assert np.array_equal(bits_of(outs[0]), bits_of(outs[1]))
    check_attention(f64_of(outs[0]), orc.decode_attention(F64(q), F64(kc_h), F64(vc_h)), f"decode {hq}/{hkv} d={d} n={n0 + 1}")


MANY = 2 ** 31 - 1   # looks: as many as the library's bound


def decode_attn_with_looks(plan, q, kc, vc, n, looks, ws=None):
    """purekv_decode_attn with a bound of its own on the gathering workgroups' looks (csrc/testing.h).  ws: the workspace to use
    (default: the plan's)."""
    nb, cap, out = plan.workspace_bytes(pk.OP_DECODE, cap=kc.shape[-2]), kc.shape[-2], torch.empty_like(q)
    ws = plan._n.workspace(pk.OP_DECODE, nb, q, 0, 0, cap) if ws is None else ws
    fn, p = pk.raw().purekv_testing_decode_attn, ctypes.c_void_p
    fn.argtypes = [p, p, p, p, ctypes.c_int32, ctypes.c_int32, p, p, ctypes.c_size_t, ctypes.c_int32, p]
    assert fn(plan.handle, q.data_ptr(), kc.data_ptr(), vc.data_ptr(), n, cap, out.data_ptr(), ws.data_ptr(), nb, looks,
              torch.cuda.current_stream().cuda_stream) == pk.OK
    return out


@pytest.mark.parametrize("hq,hkv,d,ns", [
    (28, 4, 128, (128, 129, 256, 257)),     # one chunk of 128, of 256, the first cut caches
    (28, 4, 128, (57 * 128, 57 * 128 + 1)),  # 256 compute units hold 57 chunks per KV head beside 28 gathering workgroups
    (8, 8, 64, (31 * 256, 31 * 256 + 1, 64 * 512 + 1)),   # chunks of 256, then 512; a second pass over 65 chunks
    (300, 1, 64, (600,)),                   # more heads than compute units: 19 head blocks, the last with 12 heads
    (5, 5, 128, (300,)),                    # one query head a KV head: one gathering workgroup each
])
def test_decode_gathers_chunks_of_every_size(hq, hkv, d, ns):
    """Chunks of 128, 256 and 512 keys, added up by the gathering workgroups or, where these look once or not at all, by the last
    one: the same bits, against the oracle.  All on one workspace, with another query and another cache for every length and back:
    a partial result of an earlier call that was left or read again would be of other numbers.  Every call leaves the
    workspace at zero, which is what tells a written word, and touches nothing behind it."""
    from workloads import f32_to_bf16_bits
    rng = np.random.default_rng(hq + ns[0])
    cap = max(ns)
    plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
    nb = plan.workspace_bytes(pk.OP_DECODE, cap=cap)
    ws = torch.full((nb + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    assert pk.raw().purekv_workspace_init(plan.handle, pk.OP_DECODE, ws.data_ptr(), nb, 0, 0, cap,
                                          torch.cuda.current_stream().cuda_stream) == pk.OK
    for n in (*ns, *reversed(ns)):
        q, k, v = (f32_to_bf16_bits(rng.standard_normal((x, y, d)).astype(np.float32)) for x, y in ((hq, 1), (hkv, cap), (hkv, cap)))
        v[:, ::7] = 0    # partial outputs that are exactly zero
        v[:, :, 5] = 0
        qd, kd, vd = to_dev(q[:, 0]), to_dev(k), to_dev(v)
        outs = []
        for looks in (MANY, 0, 1, MANY):
            outs.append(bits_of(decode_attn_with_looks(plan, qd, kd, vd, n, looks, ws)))
            assert not ws[:nb].any() and (ws[nb:] == 0xA5).all(), f"{hq}/{hkv} n={n} looks={looks}"
        assert all(np.array_equal(outs[0], o) for o in outs[1:]), f"{hq}/{hkv} n={n}"
        check_attention(f64_of(torch.from_numpy(outs[0].view(np.int16)).view(torch.bfloat16)),
                        orc.decode_attention(F64(q[:, 0]), F64(k[:, :n]), F64(v[:, :n])), f"decode {hq}/{hkv} d={d} n={n}")


@pytest.mark.parametrize("hq,hkv,d,n", [(28, 4, 128, 5491), (28, 4, 128, 6900), (16, 2, 64, 4000), (28, 4, 128, 16000)])
def test_decode_is_gathered_by_the_workgroups_that_wait(hq, hkv, d, n):
    """Results are the same whoever adds them up, so only the time tells that the gathering workgroups do: the last workgroup alone
    takes two to three times as long, and looks at registers instead of memory would all be used up first (0.1 ms)."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
    q, k, v = (torch.randn(x, generator=gen, device="cuda").bfloat16() for x in ((hq, d), (hkv, n, d), (hkv, n, d)))
    waits, alone = (_graph_us(lambda: decode_attn_with_looks(plan, q, k, v, n, looks)) for looks in (MANY, 0))
    print(f"[case] decode {hq}/{hkv} heads of {d}, {n} keys: {waits:.2f} us, {alone:.2f} without waiting", flush=True)
    assert waits <= 0.75 * alone


@pytest.mark.parametrize("n", [192, 448, 960, 3904, 8064, 14336])
def test_decode_divides_by_the_sum(n):
    """Equal scores and whole-numbered values: sums of probabilities and of values are exact, so an output is the quotient of two whole
    numbers rounded to fp32 and then to bf16.  Quotients half way between two bf16 numbers (1 + odd / 256) tell a division from a
    product with the reciprocal, which lands beside the middle."""
    d, k = 128, n // 64                                    # n = 64 k: the sum of column c is n (1 + (2 c + 1) / 256) = 64 k + k (2 c + 1) / 4
    v = np.ones((n, d))
    c = 2 * np.arange(d) + 1
    extra = (n * c) // 256                                 # the whole part; the rest, in quarters, goes to the last key
    for j in range(n - 1):
        take = np.minimum(extra, 127)                      # 1 + 127 = 128: every value has eight significant bits
        v[j] += take
        extra = extra - take
    v[n - 1] += (n * c) % 256 / 256
    assert not extra.any() and np.array_equal(v.sum(0) * 256, n * (256.0 + c))
    vt = torch.from_numpy(v[None]).bfloat16()
    assert np.array_equal(vt.double().numpy()[0], v)
    plan = pk.Plan(1, 4, 4, 4, 2, 1, d, 3)
    gen = torch.Generator(device="cuda").manual_seed(n)
    key = torch.randn((1, n, d), generator=gen, device="cuda").bfloat16()
    out = pk.purekv_decode_attn(plan, torch.zeros((2, d), dtype=torch.bfloat16, device="cuda"), key, vt.cuda(), n)
    assert torch.equal(out.cpu(), torch.from_numpy(1 + c / 256).bfloat16().expand(2, d))


@pytest.mark.parametrize("hq,hkv,d,shorter,longer", [(2, 1, 64, 31000, 33000), (2, 1, 128, 31000, 33000), (4, 2, 128, 16000, 16384)])
def test_decode_of_a_shorter_cache_takes_no_longer(hq, hkv, d, shorter, longer):
    """Few KV heads are not cut into as many chunks as there are compute units for: a gathering workgroup takes 64 at a time.
    (Without that the shorter caches took 1.11 to 1.29 times as long as the longer ones, now 0.91 to 0.94; test_host_boundary.py
    pins the chunks, this the results and, with room for a look more or less, the time.)"""
    gen = torch.Generator(device="cuda").manual_seed(d)
    plan, times = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3), []
    q = torch.randn((hq, d), generator=gen, device="cuda").bfloat16()
    for n in (shorter, longer):
        k, v = (torch.randn((hkv, n, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
        out = torch.empty_like(q)
        times.append(_graph_us(lambda: pk.purekv_decode_attn(plan, q, k, v, n, out=out)))
        check_attention(f64_of(out), orc.decode_attention(*(F64(bits_of(x)) for x in (q, k, v))), f"decode {hq}/{hkv} d={d} n={n}")
    print(f"[case] decode {hq}/{hkv} heads of {d}: {shorter} keys {times[0]:.2f} us, {longer} {times[1]:.2f}", flush=True)
    assert times[0] <= 1.2 * times[1]


@pytest.mark.parametrize("hq,hkv,d,n0", [(2, 1, 64, 64 * 256 + 40), (2, 1, 128, 128 * 256 + 40), (2, 1, 64, 700)])
def test_decode_step_with_scores_of_minus_infinity(hq, hkv, d, n0):
    """Keys whose scores overflow to -inf have no weight, also where they fill every chunk of the final merge's first pass
    (64 chunks of 64-wide heads, 128 of 128-wide ones)."""
    from workloads import f32_to_bf16_bits
    rng = np.random.default_rng(n0)
    q, kn, vn = (rng.standard_normal((x, d)).astype(np.float32) for x in (hq, hkv, hkv))
    kc, vc = (rng.standard_normal((hkv, n0 + 1, d)).astype(np.float32) for _ in range(2))
    q[:, 0] = 2.0 ** 100
    kc[:, :, 0], kn[:, 0] = -2.0 ** 100, 0.0
    kc[:, n0 - 39:, 0] = 0.0
    q, kn, vn, kc, vc = (f32_to_bf16_bits(x) for x in (q, kn, vn, kc, vc))
    plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
    out = pk.purekv_decode_step(plan, to_dev(q), to_dev(kn), to_dev(vn), to_dev(kc), to_dev(vc), n0)
    torch.cuda.synchronize()
    kc[:, n0], vc[:, n0] = kn, vn
    check_attention(f64_of(out), orc.decode_attention(F64(q), F64(kc), F64(vc)), f"-inf scores d={d} n={n0 + 1}")


def test_tiny_config_end_to_end_chain():
    """Config 1: importance from the dense pass, ST-SpAttn prefill, V-norm top-h at ratio 0.2, compaction, one
    decode step -- every stage fed by the GPU's own previous stage and compared with the oracle's chain."""
    wl = WORKLOADS["tiny_4f"]
    inp = generate(wl)
    n, w = wl.n_tokens, wl.window
    h = pk.purekv_budget(n, w, 0.2)
    assert h == orc.budget(n, w, 0.2) == 25
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    dense, st = _plan(wl, 0), _plan(wl, 3)
    _, lse = pk.purekv_st_spattn_prefill(dense, q, k, v, want_lse=True)
    c = pk.purekv_lowlayer_importance(dense, q, k, lse, w)
    out = pk.purekv_st_spattn_prefill(st, q, k, v)
    idx = pk.purekv_topk_select(st, c, v, w, h)
    kc, vc = pk.purekv_kv_compact(st, k, v, idx, cap=h + w + 1)
    n1 = pk.purekv_kv_append(st, to_dev(inp.k_new[0]), to_dev(inp.v_new[0]), kc, vc, h + w)
    o_dec = pk.purekv_decode_attn(st, to_dev(inp.q_new[0]), kc, vc, n1)
    torch.cuda.synchronize()

    qf, kf, vf = F64(inp.q), F64(inp.k), F64(inp.v)
    c_ref = orc.window_column_sums(qf, kf, wl.n_frames, wl.patches, wl.n_text, 0, w)
    s_ref = orc.vnorm_scores(c_ref, vf)
    idx_ref = orc.topk_select(s_ref, h, n, w)
    out_ref, _ = orc.masked_attention(qf, kf, vf, wl.n_frames, wl.patches, wl.n_text, 3)
    check_attention(f64_of(out), out_ref, "chain prefill")
    assert np.all(np.abs(f64_of(c) - c_ref) <= IMPORTANCE_REL * np.maximum(c_ref, 1e-12))
    idx_g = idx.cpu().numpy()
    check_kept_sets(idx_g, idx_ref, s_ref, h)
    kr, vr = orc.compact(inp.k, inp.v, idx_g)  # bit-exact given the indices the GPU chose
    assert np.array_equal(bits_of(kc)[:, :h + w], kr) and np.array_equal(bits_of(vc)[:, :h + w], vr)
    kcat = np.concatenate([F64(kr), F64(inp.k_new[0])[:, None]], 1)
    vcat = np.concatenate([F64(vr), F64(inp.v_new[0])[:, None]], 1)
    check_attention(f64_of(o_dec), orc.decode_attention(F64(inp.q_new[0]), kcat, vcat), "chain decode")


def test_gpu_argument_errors():
    wl = WORKLOADS["tiny_4f"]
    plan = _plan(wl, 3)
    inp = generate(wl)
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    lib = pk.raw()
    c = torch.zeros((1, 256), dtype=torch.float32, device="cuda")
    idx = torch.zeros((1, 57), dtype=torch.int32, device="cuda")
    P = lambda t: t.data_ptr()  # noqa: E731
    assert lib.purekv_lowlayer_importance(plan.handle, P(q), P(k), P(c), 0, P(c), None, 0, None) == pk.EINVAL
    assert lib.purekv_lowlayer_importance(plan.handle, P(q), P(k), P(c), 289, P(c), None, 0, None) == pk.EINVAL
    assert lib.purekv_topk_select(plan.handle, P(c), None, 0, 1, 32, 257, P(idx), None, None, 0, None) == pk.EINVAL
    assert lib.purekv_topk_select(plan.handle, P(c), P(v), 0, 1, 32, 25, P(idx), None, None, 0, None) == pk.EWORKSPACE
    assert lib.purekv_topk_select(plan.handle, P(c), None, 0, 2, 32, 25, P(idx), None, None, 0, None) == pk.EINVAL
    assert lib.purekv_kv_compact(plan.handle, P(k), P(v), 0, 1, P(idx), 57, P(k), P(v), 56, None) == pk.EINVAL
    assert lib.purekv_kv_append(plan.handle, P(k), P(v), P(k), P(v), 57, 57, None) == pk.EINVAL
    assert lib.purekv_decode_attn(plan.handle, P(q), P(k), P(v), 0, 57, P(q), P(c), 1 << 20, None) == pk.EINVAL
    assert lib.purekv_decode_attn(plan.handle, P(q), P(k), P(v), 57, 57, P(q), None, 0, None) == pk.EWORKSPACE
    assert lib.purekv_decode_step(plan.handle, P(q), P(k), P(v), P(k), P(v), 57, 57, P(q), P(c), 1 << 20, None) == pk.EINVAL
    assert lib.purekv_decode_step(plan.handle, P(q), None, P(v), P(k), P(v), 5, 57, P(q), P(c), 1 << 20, None) == pk.EINVAL
    assert lib.purekv_decode_step(plan.handle, P(q), P(k), P(v), P(k), P(v), 5, 57, P(q), None, 0, None) == pk.EWORKSPACE
    dense_plan = _plan(wl, 0)
    for bad in (pk.Stack(0, 0, 1, 32, 25), pk.Stack(4, 2, 2, 32, 25), pk.Stack(4, 1, 5, 32, 25), pk.Stack(4, 1, 2, 0, 25),
                pk.Stack(4, 1, 2, 32, 257)):
        assert lib.purekv_stack_layer(dense_plan.handle, plan.handle, ctypes.byref(bad), 0, P(q), P(k), P(v), P(q), P(c),
                                      P(c), None, 0, None) == pk.EINVAL
    good = pk.Stack(4, 1, 2, 32, 25)
    args = (P(q), P(k), P(v), P(q), P(c), P(c), None, 0, None)
    assert lib.purekv_stack_layer(plan.handle, plan.handle, ctypes.byref(good), 0, *args) == pk.EINVAL   # not dense
    assert lib.purekv_stack_layer(dense_plan.handle, None, ctypes.byref(good), 3, *args) == pk.EINVAL    # needs ST plan
    assert lib.purekv_stack_layer(dense_plan.handle, plan.handle, ctypes.byref(good), 4, *args) == pk.EINVAL
    assert lib.purekv_stack_layer(dense_plan.handle, plan.handle, ctypes.byref(good), 0, P(q), P(k), P(v), P(q), None,
                                  P(c), None, 0, None) == pk.EINVAL   # a layer that emits C needs the LSE scratch
    assert lib.purekv_stack_select_compact(dense_plan.handle, plan.handle, ctypes.byref(good), P(c), P(k), P(v), 0, P(idx),
                                           P(k), P(v), 57, None, 0, None) == pk.EINVAL   # four layers need a layer stride
    assert lib.purekv_workspace_init(plan.handle, 9, None, 0, 0, 0, 0, None) == pk.EINVAL
    assert lib.purekv_workspace_init(plan.handle, pk.OP_DECODE, None, 0, 0, 0, 57, None) == pk.EWORKSPACE
    assert lib.purekv_workspace_init(plan.handle, pk.OP_COMPACT, None, 0, 0, 0, 0, None) == pk.OK   # needs none
    assert lib.purekv_calib_mfma(plan.handle, 3, 0, 10, P(c), P(c), None) == pk.EINVAL
    assert lib.purekv_calib_mfma(plan.handle, 0, 0, 0, P(c), P(c), None) == pk.EINVAL
    assert lib.purekv_calib_mfma(plan.handle, 0, 0, 10, None, P(c), None) == pk.EINVAL
    long = pk.Plan.for_workload(SMALL["longtext_2f"], 3)
    assert long.workspace_bytes(pk.OP_PREFILL) > 0
    assert lib.purekv_st_spattn_prefill(long.handle, P(q), P(k), P(v), P(q), None, None, 0, None) == pk.EWORKSPACE
    assert lib.purekv_workspace_init(long.handle, pk.OP_PREFILL, None, 0, 0, 0, 0, None) == pk.EWORKSPACE
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("mix", [0, 1, 2])
def test_calibration_loop_runs_and_reports_its_clock(mix):
    """The board-calibration loop is not part of the method: it has to run on the plan's grid, write every sink
    element with a finite value and report a plausible shader clock."""
    plan = _plan(WORKLOADS["tiny_4f"], 3)
    n_wg = plan.counts()["n_workgroups"]
    sink = torch.full((512 * n_wg,), float("nan"), dtype=torch.float32, device="cuda")
    for rnd in (False, True):
        flops, ticks = pk.purekv_calib_mfma(plan, mix, rnd, 200, sink=sink)
        torch.cuda.synchronize()
        assert flops == 2.0 * 32 * 32 * 16 * 16 * 200 * 8 * n_wg
        assert bool(torch.isfinite(sink).all())
        cyc, ref = ticks.tolist()
        assert cyc >= 200 * 16 * 32 and ref > 0          # an MFMA of this shape holds the pipe 32 cycles
        assert 0.05 < cyc / ref / 10.0 < 3.0             # GHz


@pytest.mark.parametrize("clie,st_layer,layers", [(1, 3, 5), (0, 1, 3), (2, 3, 3)])
def test_layer_stack_matches_oracle(clie, st_layer, layers):
    """Layer stack: dense layers below st_layer, ST-SpAttn from there on; layers <= clie emit column sums, a
    layer below clie is selected with its own, the rest with layer clie's and their own V; one batched
    selection and one compaction for the whole stack.  Every layer has data of its own (seed = 40 + layer)."""
    wl = SMALL["straddle_3f"]
    n, w, hkv, d = wl.n_tokens, wl.window, wl.n_kv_heads, wl.head_dim
    h = orc.budget(n, w, 0.3)
    data = [generate(wl, seed=40 + l) for l in range(layers)]
    dense, st = _plan(wl, 0), _plan(wl, 3)
    stack = pk.Stack(layers, clie, st_layer, w, h)
    k_all = torch.stack([to_dev(x.k) for x in data])
    v_all = torch.stack([to_dev(x.v) for x in data])
    lse = torch.empty((wl.n_q_heads, n), dtype=torch.float32, device="cuda")
    c_all = torch.full((clie + 1, hkv, n - w), float("nan"), dtype=torch.float32, device="cuda")
    outs = []
    for l, x in enumerate(data):
        q = to_dev(x.q)
        outs.append(pk.purekv_stack_layer(dense, st if st_layer < layers else None, stack, l, q, k_all[l], v_all[l],
                                          torch.empty_like(q), lse, c_all))
    cap = h + w + 2
    idx_all = torch.empty((layers, hkv, h + w), dtype=torch.int32, device="cuda")
    kc_all = torch.zeros((layers, hkv, cap, d), dtype=torch.bfloat16, device="cuda")
    vc_all = torch.zeros_like(kc_all)
    pk.purekv_stack_select_compact(dense, st, stack, c_all, k_all, v_all, idx_all, kc_all, vc_all)
    torch.cuda.synchronize()

    c_ref = []
    for l, x in enumerate(data):
        qf, kf, vf = F64(x.q), F64(x.k), F64(x.v)
        pattern = orc.stack_pattern(l, st_layer)
        ref, _ = orc.masked_attention(qf, kf, vf, wl.n_frames, wl.patches, wl.n_text, pattern)
        check_attention(f64_of(outs[l]), ref, f"stack layer {l} pattern {pattern}")
        if l <= clie:
            c_ref.append(orc.window_column_sums(qf, kf, wl.n_frames, wl.patches, wl.n_text, 0, w))
            got = f64_of(c_all[l])
            assert np.all(np.abs(got - c_ref[l]) <= IMPORTANCE_REL * np.maximum(np.abs(c_ref[l]), 1e-12))
    idx_ref = orc.stack_selection(c_ref, [F64(x.v) for x in data], clie, h, n, w)
    for l, x in enumerate(data):
        s_ref = orc.vnorm_scores(c_ref[min(l, clie)], F64(x.v))
        got = idx_all[l].cpu().numpy()
        check_kept_sets(got, idx_ref[l], s_ref, h)
        kr, vr = orc.compact(x.k, x.v, got)   # compaction is a bit copy of what the GPU selected
        assert np.array_equal(bits_of(kc_all[l])[:, :h + w], kr) and np.array_equal(bits_of(vc_all[l])[:, :h + w], vr)
        assert not bits_of(kc_all[l])[:, h + w:].any()


@pytest.mark.parametrize("rows", [32, 64])
def test_tile_step_skeleton_runs(rows):
    """Second calibration loop: runs on the plan's grid, fills the sink with finite values, reports its clock,
    refuses bad arguments."""
    plan = _plan(WORKLOADS["tiny_4f"], 3)
    n_wg = plan.counts()["n_workgroups"]
    src = torch.randn(2 << 20, device="cuda").to(torch.bfloat16)   # 4 MiB
    sink = torch.full((512 * n_wg,), float("nan"), dtype=torch.float32, device="cuda")
    flops, ticks = pk.purekv_calib_tile_step(plan, rows, 50, src, sink=sink)
    torch.cuda.synchronize()
    assert flops == 4.0 * 256 * 64 * 128 * 50 * n_wg
    assert bool(torch.isfinite(sink[: (512 // (rows // 32)) * n_wg]).all())
    cyc, ref = ticks.tolist()
    assert cyc >= 50 * 32 * 32 and ref > 0 and 0.05 < cyc / ref / 10.0 < 3.0
    lib = pk.raw()
    P = lambda t: t.data_ptr()  # noqa: E731
    assert lib.purekv_calib_tile_step(plan.handle, 48, 50, P(src), P(sink), P(ticks), None) == pk.EINVAL
    assert lib.purekv_calib_tile_step(plan.handle, 32, 0, P(src), P(sink), P(ticks), None) == pk.EINVAL
    assert lib.purekv_calib_tile_step(plan.handle, 32, 50, None, P(sink), P(ticks), None) == pk.EINVAL
    with pytest.raises(ValueError):
        pk.purekv_calib_tile_step(plan, 32, 50, src[:1000])


@pytest.mark.parametrize("name,patterns", [
    ("longtext_2f", [3, 1]),                         # split text rows: the combination must leave the other head alone
    ("heads7_3f", [1, 2, 1, 2, 3, 3, 0]),            # all four patterns inside one KV group
    ("heads3_4f", [2, 2, 1, 1, 1, 2]),               # d = 64, two KV heads
    ("heads3_4f", [1, 1, 1, 3, 3, 3]),               # whole KV groups: the subset plans keep the stacked shape
    ("manyunits_g7", [3] * 7 + [1] * 14 + [2] * 7 + [0] * 14),   # 6 KV groups of 7 heads, split text rows
])
def test_per_head_patterns_through_head_subset_plans(name, patterns):
    """The other reading of the dual path: every query head has a pattern of its own.  One plan per pattern over
    the heads that use it, one prefill call per plan into the same output: every head must match the oracle under
    ITS pattern, and a call must not touch the rows of heads outside its plan."""
    wl = SMALL[name]
    assert len(patterns) == wl.n_q_heads
    inp = generate(wl, seed=17)
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    out = torch.full_like(q, float("nan"))
    lse = torch.full((wl.n_q_heads, wl.n_tokens), float("nan"), dtype=torch.float32, device="cuda")
    done = np.zeros(wl.n_q_heads, bool)
    for pattern in sorted(set(patterns)):
        mask = [p == pattern for p in patterns]
        plan = pk.Plan(wl.n_frames, wl.patch_h, wl.patch_w, wl.n_text, wl.n_q_heads, wl.n_kv_heads, wl.head_dim,
                       pattern, head_mask=mask)
        before = bits_of(out).copy()
        pk.purekv_st_spattn_prefill(plan, q, k, v, out=out, lse=lse)
        torch.cuda.synchronize()
        after = bits_of(out)
        untouched = ~np.array(mask)
        assert np.array_equal(after[untouched], before[untouched]), f"pattern {pattern} wrote outside its heads"
        done |= np.array(mask)
    assert done.all()
    qf, kf, vf = F64(inp.q), F64(inp.k), F64(inp.v)
    got, got_lse = f64_of(out), f64_of(lse)
    for pattern in sorted(set(patterns)):
        heads = [h for h, p in enumerate(patterns) if p == pattern]
        ref, ref_lse = orc.masked_attention(qf, kf, vf, wl.n_frames, wl.patches, wl.n_text, pattern, heads=heads)
        check_attention(got[heads], ref, f"{name} pattern {pattern} heads {heads}")   # the oracle returns the asked heads
        assert np.abs(got_lse[heads] - ref_lse).max() < 2e-3


def test_prefill_random_shapes_sweep():
    """Seeded sweep: odd frame sizes, texts from none to long, head groupings 1..7, both head sizes, every
    pattern, with and without the log-sum-exp output -- each through the kernel and against the oracle."""
    rng = np.random.default_rng(25600)
    for case in range(24):
        ph, pw = int(rng.integers(1, 14)), int(rng.integers(1, 14))
        F = int(rng.integers(1, max(2, min(10, 900 // (ph * pw)) + 1)))
        T = int(rng.choice([0, 1, 7, 33, 129, 700]))
        hkv = int(rng.choice([1, 2, 3]))
        g = int(rng.choice([1, 2, 4, 7]))
        d = int(rng.choice([64, 128]))
        pattern = int(rng.integers(0, 4))
        wl = small_variant(f"sweep{case}", n_frames=F, patch_h=ph, patch_w=pw, n_text=T, n_q_heads=hkv * g,
                           n_kv_heads=hkv, head_dim=d)
        print(f"[case] sweep {case}: F={F} P={ph}x{pw} T={T} heads {hkv * g}/{hkv} d={d} pattern={pattern}", flush=True)
        inp = generate(wl, seed=100 + case)
        plan = _plan(wl, pattern)
        q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
        out, lse = pk.purekv_st_spattn_prefill(plan, q, k, v, want_lse=True)
        out2 = pk.purekv_st_spattn_prefill(plan, q, k, v)
        torch.cuda.synchronize()
        ref, ref_lse = orc.masked_attention(F64(inp.q), F64(inp.k), F64(inp.v), F, ph * pw, T, pattern)
        check_attention(f64_of(out), ref, f"sweep {case} (lse variant)")
        check_attention(f64_of(out2), ref, f"sweep {case}")
        assert np.abs(f64_of(lse) - ref_lse).max() < 2e-3


def test_window_plan_random_shapes_sweep():
    """Seeded sweep of window plans with more units than workgroups (many heads on short sequences), so that most of
    them are divided: outputs and the window's log-sum-exp against the oracle, every other element of lse untouched,
    output bits equal to the undivided plan's where both run a row's list whole."""
    rng = np.random.default_rng(25601)
    divided = 0
    for case in range(10):
        ph, pw = int(rng.integers(4, 14)), int(rng.integers(4, 14))
        F = max(2, int(rng.integers(900, 1600)) // (ph * pw))
        T = int(rng.choice([0, 5, 40, 129]))
        hkv, g = [(8, 7), (16, 4), (12, 7)][int(rng.integers(0, 3))]
        d = int(rng.choice([64, 128]))
        pattern = int(rng.choice([0, 1, 3, 3]))
        wl = small_variant(f"wsweep{case}", n_frames=F, patch_h=ph, patch_w=pw, n_text=T, n_q_heads=hkv * g,
                           n_kv_heads=hkv, head_dim=d)
        n = wl.n_tokens
        w = int(rng.integers(1, 48))
        inp = generate(wl, seed=300 + case)
        plan, whole = pk.Plan.for_workload(wl, pattern, lse_window=w), pk.Plan.for_workload(wl, pattern)
        c = plan.counts()
        divided += c["lse_queue0"] > 0
        print(f"[case] window sweep {case}: F={F} P={ph}x{pw} T={T} heads {hkv * g}/{hkv} d={d} pattern={pattern} w={w} "
              f"N={n} lse_queue0={c['lse_queue0']}", flush=True)
        q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
        lse = torch.full((wl.n_q_heads, n), 7.5, dtype=torch.float32, device="cuda")
        out, _ = pk.purekv_st_spattn_prefill(plan, q, k, v, lse=lse)
        out_whole = pk.purekv_st_spattn_prefill(whole, q, k, v)
        torch.cuda.synchronize()
        ref, ref_lse = orc.masked_attention(F64(inp.q), F64(inp.k), F64(inp.v), F, ph * pw, T, pattern)
        check_attention(f64_of(out), ref, f"window sweep {case}")
        got = f64_of(lse)
        assert np.all(got[:, :n - w] == 7.5) and np.abs(got[:, n - w:] - ref_lse[:, n - w:]).max() < 2e-3
        if c["n_split_qtiles"] == 0 and whole.counts()["n_split_qtiles"] == 0:
            assert np.array_equal(bits_of(out), bits_of(out_whole))
    assert divided >= 5, divided   # (a plan stays whole when the window's tiles are over a quarter of the work)


def test_importance_random_shapes_sweep():
    """Seeded sweep of the column sums: window sizes from one row to the whole sequence (text rows only, video rows
    under a mask, windows that are not a multiple of the 32-row block), odd frame sizes, 1..7 heads per KV head."""
    rng = np.random.default_rng(314)
    for case in range(20):
        ph, pw = int(rng.integers(1, 12)), int(rng.integers(1, 12))
        F = int(rng.integers(1, max(2, min(8, 700 // (ph * pw)) + 1)))
        T = int(rng.choice([0, 5, 40, 130, 300]))
        hkv = int(rng.choice([1, 2]))
        g = int(rng.choice([1, 3, 7]))
        d = int(rng.choice([64, 128]))
        pattern = int(rng.integers(0, 4))
        n = F * ph * pw + T
        w = int(rng.choice([1, 31, 32, 33, max(1, T), max(1, n // 3), n]))
        w = min(max(w, 1), n)
        wl = small_variant(f"isweep{case}", n_frames=F, patch_h=ph, patch_w=pw, n_text=T, n_q_heads=hkv * g,
                           n_kv_heads=hkv, head_dim=d)
        print(f"[case] importance sweep {case}: N={n} w={w} heads {hkv * g}/{hkv} d={d} pattern={pattern}", flush=True)
        inp = generate(wl, seed=200 + case)
        plan = _plan(wl, pattern)
        q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
        _, lse = pk.purekv_st_spattn_prefill(plan, q, k, v, want_lse=True)
        c = pk.purekv_lowlayer_importance(plan, q, k, lse, w)
        torch.cuda.synchronize()
        ref = orc.window_column_sums(F64(inp.q), F64(inp.k), F, ph * pw, T, pattern, w)
        got = f64_of(c)
        assert got.shape == ref.shape
        if ref.size:
            rel = np.abs(got - ref) / np.maximum(np.abs(ref), 1e-12)
            assert rel.max() <= IMPORTANCE_REL, f"case {case}: worst rel {rel.max():.3g}"
            assert np.all(got[ref == 0] == 0)


def test_decode_random_shapes_sweep():
    """Seeded sweep of the decode step: cache lengths around the 32-key wavefront tiles and the 256-key chunks, 1 to
    20 query heads per KV head (more than one block of 16), both head sizes; fused append + attention against the
    oracle on the grown cache, and the cache rows themselves."""
    from workloads import f32_to_bf16_bits
    rng = np.random.default_rng(77)
    for case in range(24):
        hkv = int(rng.choice([1, 2, 5]))
        g = int(rng.choice([1, 2, 7, 16, 17, 20]))
        d = int(rng.choice([64, 128]))
        n0 = int(rng.choice([0, 1, 15, 16, 31, 32, 33, 255, 256, 257, 511, 513, 1000, 2049]))
        hq = hkv * g
        bits = lambda *shape: f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))  # noqa: E731
        cap = n0 + 3
        kc_h, vc_h = bits(hkv, cap, d), bits(hkv, cap, d)
        kc, vc = to_dev(kc_h), to_dev(vc_h)
        plan = pk.Plan(1, 4, 4, 4, hq, hkv, d, 3)
        print(f"[case] decode sweep {case}: heads {hq}/{hkv} d={d} n0={n0}", flush=True)
        for t in range(2):
            q, kn, vn = bits(hq, d), bits(hkv, d), bits(hkv, d)
            out = pk.purekv_decode_step(plan, to_dev(q), to_dev(kn), to_dev(vn), kc, vc, n0 + t)
            torch.cuda.synchronize()
            kc_h[:, n0 + t], vc_h[:, n0 + t] = kn, vn
            assert np.array_equal(bits_of(kc), kc_h) and np.array_equal(bits_of(vc), vc_h)
            ref = orc.decode_attention(F64(q), F64(kc_h)[:, :n0 + t + 1], F64(vc_h)[:, :n0 + t + 1])
            check_attention(f64_of(out), ref, f"decode sweep {case} step {t}")


def test_two_streams_share_one_plan():
    """A plan holds no mutable device state: decode calls and prefill calls (with split lists) on two streams, each
    with a workspace of its own, may overlap on the GPU.  Both streams' results against the oracle, several rounds."""
    wl = SMALL["heads7_3f"]          # text rows split into slices: the prefill hands partial results over in its workspace
    n, hq, hkv, d = wl.n_tokens, wl.n_q_heads, wl.n_kv_heads, wl.head_dim
    plan = _plan(wl, 3)
    assert plan.counts()["n_split_qtiles"] > 0
    data = [generate(wl, seed=80 + i, decode_steps=1) for i in range(2)]
    n_c = 1100                       # five chunks of cached keys: the decode kernel merges through its workspace
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    dev = [[to_dev(x) for x in (dt.q, dt.k, dt.v, dt.q_new[0])] for dt in data]
    torch.cuda.synchronize()
    outs, decs = [[], []], [[], []]
    for rnd in range(6):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                q, k, v, qn = dev[i]
                outs[i].append(pk.purekv_st_spattn_prefill(plan, q, k, v))
                decs[i].append(pk.purekv_decode_attn(plan, qn, k[:, :n_c].contiguous(), v[:, :n_c].contiguous(), n_c))
    torch.cuda.synchronize()
    for i, dt in enumerate(data):
        ref, _ = orc.masked_attention(F64(dt.q), F64(dt.k), F64(dt.v), wl.n_frames, wl.patches, wl.n_text, 3)
        dref = orc.decode_attention(F64(dt.q_new[0]), F64(dt.k)[:, :n_c], F64(dt.v)[:, :n_c])
        for rnd in range(6):
            check_attention(f64_of(outs[i][rnd]), ref, f"stream {i} round {rnd} prefill")
            check_attention(f64_of(decs[i][rnd]), dref, f"stream {i} round {rnd} decode")
            assert np.array_equal(bits_of(outs[i][rnd]), bits_of(outs[i][0]))   # and reproducible bit for bit
            assert np.array_equal(bits_of(decs[i][rnd]), bits_of(decs[i][0]))


def test_calls_from_inside_a_workspace_allocation():
    """A dispatch mode sees the allocation of a workspace and calls the same plan on other streams meanwhile: their
    buffers enter the plan's list while the outer call is about to replace its own, which was too small."""
    from torch.utils._python_dispatch import TorchDispatchMode
    wl = SMALL["heads7_3f"]
    plan, again = _plan(wl, 3), _plan(wl, 3)
    hq, hkv, d = wl.n_q_heads, wl.n_kv_heads, wl.head_dim
    gen = torch.Generator(device="cuda").manual_seed(4)
    q = torch.randn((hq, d), generator=gen, device="cuda").bfloat16()
    short, long = (torch.randn((2, hkv, n, d), generator=gen, device="cuda").bfloat16() for n in (600, 5000))
    out = torch.empty_like(q)
    streams = [torch.cuda.Stream() for _ in range(12)]
    want_short, want_long = (pk.purekv_decode_attn(again, q, x[0], x[1], x.shape[2]) for x in (short, long))
    pk.purekv_decode_attn(plan, q, short[0], short[1], 600, out=out)
    torch.cuda.synchronize()
    inner, empties = [], []

    class Reenter(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            if func._schema.name.startswith("aten::empty"):
                empties.append(tuple(args[0]))
                if not inner:
                    for s in streams:
                        with torch.cuda.stream(s):
                            inner.append(pk.purekv_decode_attn(plan, q, short[0], short[1], 600))
            return func(*args, **(kwargs or {}))

    with Reenter():
        pk.purekv_decode_attn(plan, q, long[0], long[1], 5000, out=out)
    torch.cuda.synchronize()
    assert len(inner) == len(streams) and torch.equal(out, want_long)
    assert all(torch.equal(x, want_short) for x in inner)
    # every buffer is in the list: nothing is allocated again
    n = len(empties)
    with Reenter():
        pk.purekv_decode_attn(plan, q, long[0], long[1], 5000, out=out)
        for s, x in zip(streams, inner):
            with torch.cuda.stream(s):
                pk.purekv_decode_attn(plan, q, short[0], short[1], 600, out=x)
    torch.cuda.synchronize()
    assert len(empties) == n and torch.equal(out, want_long) and all(torch.equal(x, want_short) for x in inner)


def test_an_output_that_does_not_fit_raises_out_of_memory():
    wl = SMALL["heads3_4f"]
    inp = generate(wl, seed=3)
    plan = _plan(wl, 3)
    k, v = to_dev(inp.k), to_dev(inp.v)
    idx = torch.arange(40, dtype=torch.int32, device="cuda").repeat(wl.n_kv_heads, 1)
    cap = 2 ** 31 - 1
    assert wl.n_kv_heads * cap * wl.head_dim * 2 > torch.cuda.mem_get_info()[1]
    with pytest.raises(torch.OutOfMemoryError):
        pk.purekv_kv_compact(plan, k, v, idx, cap=cap)
    kc, vc = pk.purekv_kv_compact(plan, k, v, idx)
    assert torch.equal(kc, k[:, :40]) and torch.equal(vc, v[:, :40])


def test_two_threads_grow_one_workspace():
    """Two threads on one stream and one plan whose decode calls need larger and larger workspaces: a buffer that one
    thread replaces stays alive until the other's launch is queued.  Bit-equal to the same calls from one thread."""
    wl = SMALL["heads7_3f"]
    plan, again = _plan(wl, 3), _plan(wl, 3)
    hq, hkv, d = wl.n_q_heads, wl.n_kv_heads, wl.head_dim
    gen = torch.Generator(device="cuda").manual_seed(9)
    kv = torch.randn((2, hkv, 6000, d), generator=gen, device="cuda").bfloat16()
    q = torch.randn((hq, d), generator=gen, device="cuda").bfloat16()
    sizes = [300 + 257 * i for i in range(20)]
    caches = [(kv[0, :, :n].contiguous(), kv[1, :, :n].contiguous()) for n in sizes]
    want = [pk.purekv_decode_attn(again, q, k, v, n) for n, (k, v) in zip(sizes, caches)]
    got = [[None] * len(sizes) for _ in range(2)]

    def work(t):
        for i, (n, (k, v)) in enumerate(zip(sizes, caches)):
            got[t][i] = pk.purekv_decode_attn(plan, q, k, v, n)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for t in range(2):
        for i in range(len(sizes)):
            assert torch.equal(got[t][i], want[i]), f"thread {t}, {sizes[i]} keys"


@pytest.mark.parametrize("pattern", [0, 3])
@pytest.mark.parametrize("name", ["tiny_4f", "ragged_3f", "straddle_3f", "heads7_3f", "heads3_4f", "manyunits_g7",
                                  "manyunits_g1", "single_token", "longtext_2f"])
def test_prefill_emits_squared_v_norms(name, pattern):
    """The V-norm weighting without a second pass over V (Eq. 3 / Eq. 4): the prefill call that also emits
    ||v_j||^2 for every key writes every entry exactly once (NaN-filled buffer), equal to the oracle's norms, and
    leaves the attention output bit for bit what the plain call gives; the selection from C and these norms is the
    oracle's."""
    wl = SMALL[name]
    inp = generate(wl, seed=33)
    n, w = wl.n_tokens, min(wl.window if wl.window else 1, wl.n_tokens)
    w = max(w, 1)
    print(f"[case] prefill+vnorm {name} pattern={pattern}", flush=True)
    plan = _plan(wl, pattern)
    q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v)
    out_plain, lse_plain = pk.purekv_st_spattn_prefill(plan, q, k, v, want_lse=True)
    vn2 = torch.full((wl.n_kv_heads, n), float("nan"), dtype=torch.float32, device="cuda")
    out, lse = pk.purekv_st_spattn_prefill(plan, q, k, v, want_lse=True, vnorm2=vn2)
    out_nolse = pk.purekv_st_spattn_prefill(plan, q, k, v, vnorm2=torch.empty_like(vn2))
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(out), bits_of(out_plain)) and torch.equal(lse, lse_plain)
    assert np.array_equal(bits_of(out_nolse), bits_of(out_plain))
    vf = F64(inp.v)
    ref = (vf * vf).sum(2)
    got = f64_of(vn2)
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - ref) <= 2e-6 * ref + 1e-30), f"worst rel {np.max(np.abs(got - ref) / np.maximum(ref, 1e-30)):.3g}"
    if n - w >= 1:
        h = max(1, orc.budget(n, w, 0.3)) if n - w >= 2 else 1
        h = min(h, n - w)
        c = np.random.default_rng(5).random((wl.n_kv_heads, n - w)).astype(np.float32)
        idx, s = pk.purekv_topk_select_vnorm(plan, torch.from_numpy(c).cuda(), vn2, w, h, want_scores=True)
        idx2 = pk.purekv_topk_select_vnorm(plan, torch.from_numpy(c).cuda(), vn2, w, h)   # workspace path
        torch.cuda.synchronize()
        assert torch.equal(idx, idx2)
        s_ref = orc.vnorm_scores(c.astype(np.float64), vf)
        assert np.all(np.abs(f64_of(s) - s_ref) <= 2e-6 * np.abs(s_ref) + 1e-30)
        check_kept_sets(idx.cpu().numpy(), orc.topk_select(s_ref, h, n, w), s_ref, h)


@pytest.mark.parametrize("hq,hkv,d,frames,patch,text,pattern", [
    (16, 2, 128, 8, 10, 96, 0), (8, 8, 128, 8, 17, 100, 0), (32, 8, 128, 8, 10, 96, 3), (4, 2, 64, 8, 10, 96, 3)])
def test_v_norms_cost_a_short_pass_where_few_wavefronts_have_rows(hq, hkv, d, frames, patch, text, pattern):
    """Plans of four wavefronts or fewer a workgroup take the norms from a pass over V (2.3 us here), not from the launch, whose
    steps wait for them there (12 to 18 us with heads of 128); bit for bit the norms that any such plan's call gives.  With heads of
    64 and three wavefronts or fewer the launch emits them (0 to 3 us); their sums are added up in another order."""
    plan = pk.Plan(frames, patch, patch, text, hq, hkv, d, pattern)
    n, c = plan.N, plan.counts()
    assert c["stacked_heads"] * c["row_blocks"] <= pk.WAVES // 2
    gen = torch.Generator(device="cuda").manual_seed(n + hq)
    q, k, v = (torch.randn((x, n, d), generator=gen, device="cuda").bfloat16() for x in (hq, hkv, hkv))
    out, n2 = plan.empty_out("cuda"), torch.full((hkv, n), float("nan"), dtype=torch.float32, device="cuda")
    plain = _graph_us(lambda: pk.purekv_st_spattn_prefill(plan, q, k, v, out=out))
    norms = _graph_us(lambda: pk.purekv_st_spattn_prefill(plan, q, k, v, out=out, vnorm2=n2))
    print(f"[case] {hq}/{hkv} heads of {d}, {n} tokens: {plain:.1f} us, with norms {norms:.1f}", flush=True)
    assert norms <= plain + 7.0
    eight = pk.Plan(1, 1, 1, n - 1, 512, hkv, d, 0)   # eight wavefronts: a pass of its own as well
    assert eight.counts()["stacked_heads"] * eight.counts()["row_blocks"] == pk.WAVES
    ref = torch.full_like(n2, float("nan"))
    big = torch.zeros((512, n, d), dtype=torch.bfloat16, device="cuda")
    pk.purekv_st_spattn_prefill(eight, big, k, v, vnorm2=ref)
    if d == 128:
        assert torch.equal(n2.view(torch.int32), ref.view(torch.int32))
    assert ((n2 - ref).abs() <= 64 * 2 ** -24 * ref).all()   # at most d additions, each within an ulp, of squares


def test_prefill_vnorm_layers_and_head_subsets():
    """Layered norms [L, Hkv, N] through one batched selection, and a plan over a head subset: the KV heads none of
    whose query heads it covers keep what the buffer held."""
    wl = SMALL["heads3_4f"]       # 6 query heads on 2 KV heads
    n, w = wl.n_tokens, wl.window
    h = orc.budget(n, w, 0.4)
    layers = [generate(wl, seed=90 + l) for l in range(3)]
    plan = _plan(wl, 3)
    vn_all = torch.empty((3, wl.n_kv_heads, n), dtype=torch.float32, device="cuda")
    for l, x in enumerate(layers):
        pk.purekv_st_spattn_prefill(plan, to_dev(x.q), to_dev(x.k), to_dev(x.v), vnorm2=vn_all[l])
    c = np.random.default_rng(6).random((wl.n_kv_heads, n - w)).astype(np.float32)
    idx = pk.purekv_topk_select_vnorm(plan, torch.from_numpy(c).cuda(), vn_all, w, h)
    v_all = torch.stack([to_dev(x.v) for x in layers])
    idx_v = pk.purekv_topk_select(plan, torch.from_numpy(c).cuda(), v_all, w, h)
    torch.cuda.synchronize()
    for l, x in enumerate(layers):
        s_ref = orc.vnorm_scores(c.astype(np.float64), F64(x.v))
        check_kept_sets(idx[l].cpu().numpy(), orc.topk_select(s_ref, h, n, w), s_ref, h)
        check_kept_sets(idx_v[l].cpu().numpy(), orc.topk_select(s_ref, h, n, w), s_ref, h)
    sub = pk.Plan(wl.n_frames, wl.patch_h, wl.patch_w, wl.n_text, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, 3,
                  head_mask=[0, 0, 0, 1, 0, 1])            # query heads 3 and 5: KV head 1 only
    x = layers[0]
    vn = torch.full((wl.n_kv_heads, n), -7.0, dtype=torch.float32, device="cuda")
    pk.purekv_st_spattn_prefill(sub, to_dev(x.q), to_dev(x.k), to_dev(x.v), vnorm2=vn)
    torch.cuda.synchronize()
    vf = F64(x.v)
    assert torch.all(vn[0] == -7.0)
    assert np.all(np.abs(f64_of(vn[1]) - (vf[1] ** 2).sum(1)) <= 2e-6 * (vf[1] ** 2).sum(1))


@pytest.mark.parametrize("n", [2, 3, 255, 256, 257, 1000, 8192, 20000])
def test_spearman_matches_oracle_exactly(n):
    """Sec. 3.3, Eq. 5-7: ranks are counts and the sum of squared rank differences an integer: bit-exact; rho is the
    correctly rounded quotient on both sides."""
    rng = np.random.default_rng(50 + n)
    rows = 5
    a = rng.standard_normal((rows, n)).astype(np.float32)
    b = (0.5 * a + rng.standard_normal((rows, n))).astype(np.float32)
    b[1] = a[1]                                                    # identical rankings
    b[2] = -a[2]                                                   # reversed
    a[3] = rng.integers(0, 4, size=n).astype(np.float32)           # heavy ties, signed zeros among them
    b[3] = rng.integers(0, 3, size=n).astype(np.float32)
    a[3, ::7] = -0.0
    b[4] = np.float32(1.5)                                         # one array constant: its ranks are the indices
    print(f"[case] spearman n={n}", flush=True)
    d2, rho = pk.purekv_spearman(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda())
    torch.cuda.synchronize()
    ref_d2, ref_rho = orc.spearman_rank_correlation(a.astype(np.float64), b.astype(np.float64))
    assert d2.cpu().numpy().tolist() == [int(x) for x in ref_d2]
    assert np.array_equal(rho.cpu().numpy(), ref_rho)
    assert rho[1].item() == 1.0
    if np.unique(a[2]).size == n:      # (two equal scores keep their index order in both arrays: not a full reversal)
        assert rho[2].item() == -1.0


def test_spearman_of_estimated_against_own_scores_through_the_library():
    """The check of Sec. 3.3 end to end on one synthetic layer pair: S-hat from the low layer's column sums and the
    high layer's V (Eq. 4), S from the high layer's own column sums (Eq. 6), both through the library, compared with
    the oracle's scores and ranks."""
    wl = SMALL["straddle_3f"]
    low, high = generate(wl, seed=31), generate(wl, seed=32)
    n, w = wl.n_tokens, wl.window
    h = pk.purekv_budget(n, w, 0.2)
    plan = pk.Plan.for_workload(wl, 0)
    scores = []
    for inp in (low, high):
        q, k, v = to_dev(inp.q), to_dev(inp.k), to_dev(high.v)
        _, lse = pk.purekv_st_spattn_prefill(plan, q, k, to_dev(inp.v), want_lse=True)
        c = pk.purekv_lowlayer_importance(plan, q, k, lse, w)
        _, s = pk.purekv_topk_select(plan, c, v, w, h, want_scores=True)
        scores.append(s.reshape(wl.n_kv_heads, n - w).contiguous())
    d2, rho = pk.purekv_spearman(scores[0], scores[1])
    torch.cuda.synchronize()
    # the oracle on the library's own fp32 scores: exact; and on its own fp64 scores: the same rho up to the few keys
    # whose order the fp32 rounding of nearly equal scores changes
    ref_d2, ref_rho = orc.spearman_rank_correlation(f64_of(scores[0]), f64_of(scores[1]))
    assert d2.cpu().numpy().tolist() == [int(x) for x in ref_d2] and np.array_equal(rho.cpu().numpy(), ref_rho)
    vf = F64(high.v)
    s_hat = orc.vnorm_scores(orc.window_column_sums(F64(low.q), F64(low.k), wl.n_frames, wl.patches, wl.n_text, 0, w), vf)
    s_own = orc.vnorm_scores(orc.window_column_sums(F64(high.q), F64(high.k), wl.n_frames, wl.patches, wl.n_text, 0, w), vf)
    _, rho64 = orc.spearman_rank_correlation(s_hat, s_own)
    assert np.abs(rho.cpu().numpy() - rho64).max() < 1e-3
    # the two layers' Q and K are independent draws here, but both score arrays carry the same V norms: the rankings
    # agree more than chance (n ~ 1700 keys: chance is |rho| < 0.08 at three sigma)
    assert (rho.cpu().numpy() > 0.08).all()


def test_spearman_argument_errors():
    a = torch.zeros((2, 8), dtype=torch.float32, device="cuda")
    out = torch.zeros(2, dtype=torch.int64, device="cuda")
    lib = pk.raw()
    assert lib.purekv_spearman(a.data_ptr(), a.data_ptr(), 2, 1, out.data_ptr(), None, None) == pk.EINVAL
    assert lib.purekv_spearman(a.data_ptr(), a.data_ptr(), 2, 131073, out.data_ptr(), None, None) == pk.EINVAL
    assert lib.purekv_spearman(a.data_ptr(), a.data_ptr(), 0, 8, out.data_ptr(), None, None) == pk.EINVAL
    assert lib.purekv_spearman(None, a.data_ptr(), 2, 8, out.data_ptr(), None, None) == pk.EINVAL
    assert lib.purekv_spearman(a.data_ptr(), a.data_ptr(), 2, 8, None, None, None) == pk.EINVAL
    assert lib.purekv_spearman(a.data_ptr(), a.data_ptr(), 2, 8, out.data_ptr(), None, None) == pk.OK   # rho is optional
    torch.cuda.synchronize()
    assert out.tolist() == [0, 0]
