"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded inputs.

Small shapes compare every unit at every step; the Janus-Pro-shaped configurations run at full size in
the benchmark's launch configuration and compare sampled units.  Index sets are compared exactly,
outputs within the stated tolerance."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2510_18716_amd as ssd
import workload
from harness import (GAP_MARGIN, ROPE_BF16_MARGIN, check_outputs, check_selection_on_own_scores, compare_unit_sets, gpu_decode,
                     make_cache, near_tie_cap, oracle_unit, rotate_rows, sample_units, say, settle_near_tie)

pytestmark = pytest.mark.gpu


def _to_cuda(data):
    return {k: v.cuda() for k, v in data.items()}


def _full_compare(wl, ht=None, lpc=None, k_units=10 ** 9, export_every=1, seed=0, device_gen=False, fused=False, rope=0,
                  accumulate=True, shape=None, split=0):
    ht = workload.head_map(wl) if ht is None else ht
    schedule = workload.compress_schedule(wl)
    say("case", wl.name, wl.dtype, "L%d B%d H%d d%d n0=%d N=%d W%d S%d M%d R%d C%d cadence%d lpc=%s fused=%s rope=%d acc=%d split=%d" % (
        wl.L, wl.B, wl.H, wl.d, wl.n0, wl.N, wl.W, wl.S, wl.M, wl.R, wl.C, wl.cadence, lpc, fused, rope, accumulate, split))
    if device_gen:
        dev_data = workload.generate(wl, device="cuda", head_type=ht)
    else:
        data = workload.generate(wl, head_type=ht)
        dev_data = _to_cuda(data)
    units = sample_units(wl, ht, k_units, seed)
    if export_every == 1:
        steps = list(range(wl.n_total))
    else:
        comp = [p for p in range(wl.n_total) if schedule[p]]
        steps = sorted(set(range(0, wl.n_total, export_every)) | {wl.n_total - 1} | set(comp[:: max(1, len(comp) // 8)]))
    outs, exports, cache = gpu_decode(wl, dev_data, ht, schedule, units, layers_per_call=lpc, export_steps=steps, fused=fused,
                                      rope=rope, accumulate=accumulate, shape=shape, split=split)
    say("  gpu decode done: %d units, %d exported steps" % (len(units), len(exports)))
    # sampled units back on the host: the oracle sees the very same bits
    layers = sorted(set(l for (l, _, _) in units))
    near_ties, worst, t3 = 0, 0.0, 0
    final_pos, final_score = exports[wl.n_total - 1]["post"]
    # scores and near-tie margin: 1e-4, except where the two sides may hold keys that differ by one bf16 rounding
    margin = ROPE_BF16_MARGIN if (rope and wl.dtype == "bf16") else GAP_MARGIN
    for ui, unit in enumerate(units):
        l, b, h = unit
        host = {x: dev_data[x][:, l:l + 1, b:b + 1, h:h + 1].cpu() for x in "qkv"}
        if rope:        # the oracle gets q and k rotated by its own routine, then takes the ordinary route
            host["q"], host["k"] = rotate_rows(wl, host["q"], rope), rotate_rows(wl, host["k"], rope)
        o_ref, hl, gl, u = oracle_unit(wl, host, ht[l:l + 1, h:h + 1], schedule, (0, 0, 0), layer=l, head=h, accumulate=accumulate)
        li = layers.index(l)
        diverged = compare_unit_sets(wl, ht, unit, li, exports, hl, gl, schedule, margin=margin)
        # the GPU's selections on its own scores, at every exported cut before a divergence (a near-tie's own
        # step is settled below; after it the unit is no longer the oracle's)
        upto_p = wl.n_total if diverged is None else diverged[0]
        t3 += len(check_selection_on_own_scores(wl, ht, unit, li, {p: e for p, e in exports.items() if p < upto_p}))
        upto = wl.n_total if diverged is None else diverged[0] + 1
        worst = max(worst, check_outputs(outs[:upto, ui], o_ref[:upto], wl.dtype, "unit %s" % (unit,)))
        if diverged is not None:
            near_ties += 1
            say("  near-tie: unit %s, cut at step %d (margin %.2e), seen at step %d" % (unit, diverged[0], gl[diverged[0]], diverged[1]))
            settle_near_tie(wl, dev_data, ht, schedule, unit, li, exports, diverged[0], fused, lpc=lpc, rope=rope, shape=shape,
                            accumulate=accumulate)
            continue
        if ht[l, h] == workload.SEMANTIC:
            hp, hs, sp, ss = u.state()
            ref = dict(zip(hp.tolist() + sp.tolist(), hs.tolist() + ss.tolist()))
            got = {int(p): float(s) for p, s in zip(final_pos[li, b, h], final_score[li, b, h]) if p >= 0}
            assert sorted(got) == sorted(ref)
            for p in ref:
                assert abs(got[p] - ref[p]) <= margin * max(1.0, abs(ref[p])), ("score", unit, p, got[p], ref[p])
    say("  max abs output error %.3e, near-tie units %d of %d, own-score selections checked %d" % (
        worst, near_ties, len(units), t3))
    assert near_ties <= near_tie_cap(len(units))
    if any(schedule[p] for p in exports) and any(ht[l, h] == workload.SEMANTIC for (l, _, h) in units):
        assert t3 > 0, "no selection was checked on the GPU's own scores"
    return cache


# ------------------------------------------------------------------ tiny, every unit, every step ----

FUSED = pytest.mark.parametrize("fused", [False, True], ids=["three-calls", "fused-step"])


@FUSED
@pytest.mark.parametrize("S,cadence", [(1, 1), (0, 1), (1, 8)])
def test_config1_every_unit_every_step(S, cadence, fused):
    wl = workload.config(1).replace(S=S, cadence=cadence, C=1 + cadence)
    _full_compare(wl, fused=fused)


@FUSED
def test_config1_plain_gaussian_inputs(fused):
    # no planted structure: every retained row carries weight, so a wrong row shows in the output
    wl = workload.config(1).replace(plain=True, name="cfg1-plain")
    _full_compare(wl, fused=fused)


@FUSED
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_small_shapes_all_dtypes(dtype, d, fused):
    wl = workload.Workload("small-%s-%d" % (dtype, d), L=3, prompts=2, H=6, d=d, dtype=dtype, n0=9, grid_h=7,
                           grid_w=9, W=13, M=10, S=2, R=2, C=7, cadence=5, spatial_frac=0.5, seed=77,
                           plain=True)
    _full_compare(wl, fused=fused)
    _full_compare(wl.replace(name=wl.name + "-perlayer"), lpc=1, fused=fused)


@FUSED
def test_ragged_sizes_and_long_row_buffer(fused):
    # row counts that are not multiples of the rows-per-load (4) or the chunk (16); a row buffer that wraps
    wl = workload.Workload("ragged", L=2, prompts=1, H=5, d=128, dtype="bf16", n0=3, grid_h=9, grid_w=11, W=67,
                           M=33, S=3, R=5, C=41, cadence=36, spatial_frac=0.4, seed=5, plain=True)
    _full_compare(wl, fused=fused)


@FUSED
def test_all_spatial_and_all_semantic_head_maps(fused):
    # the two special cases the paper compares against: window + sink tokens only, heavy hitters only
    wl = workload.Workload("all-spatial", L=2, prompts=1, H=4, d=64, dtype="bf16", n0=4, grid_h=6, grid_w=6, W=8,
                           M=6, S=1, R=1, C=2, cadence=1, seed=9, plain=True)
    _full_compare(wl, ht=np.zeros((2, 4), np.uint8), fused=fused)
    _full_compare(wl.replace(name="all-semantic"), ht=np.ones((2, 4), np.uint8), fused=fused)
    mixed = np.array([[0, 0, 0, 0], [1, 1, 1, 1]], np.uint8)      # head lists that differ per layer
    _full_compare(wl.replace(name="layerwise-types"), ht=mixed, fused=fused)


@FUSED
def test_degenerate_parameters(fused):
    base = dict(L=1, prompts=1, H=4, d=64, dtype="f32", n0=2, grid_h=5, grid_w=5, seed=3, plain=True)
    _full_compare(workload.Workload("W1-M1", W=1, M=1, S=0, R=1, C=2, cadence=1, **base), fused=fused)
    _full_compare(workload.Workload("R0", W=2, M=3, S=1, R=0, C=1, cadence=1, **base), fused=fused)
    _full_compare(workload.Workload("S-exceeds-n0", W=4, M=4, S=6, R=3, C=4, cadence=1, **base), fused=fused)


@FUSED
def test_attention_without_score_accumulation(fused):
    # accumulate_scores = 0 (Algorithm 2: scores are accumulated only "if attention scores available"): every score
    # stays 0, so each cut keeps the lowest positions; outputs, sets and the all-zero scores against the oracle on
    # the same route.  Short and long row buffers (register and general selection), both dtypes, Algorithm 2.
    wl = workload.Workload("no-acc", L=2, prompts=2, H=6, d=128, dtype="bf16", n0=9, grid_h=7, grid_w=9, W=13, M=10, S=2,
                           R=2, C=7, cadence=5, seed=91, plain=True)
    _full_compare(wl, fused=fused, accumulate=False)
    _full_compare(wl.replace(name="no-acc-cadence1", R=1, C=2, cadence=1), lpc=1, fused=fused, accumulate=False)
    _full_compare(wl.replace(name="no-acc-f32-64", dtype="f32", d=64), fused=fused, accumulate=False)
    _full_compare(wl.replace(name="no-acc-long-buffer", R=3, C=40, cadence=33), fused=fused, accumulate=False)
    _full_compare(wl.replace(name="no-acc-alg2", alg2=True, R=0, C=6, cadence=6), fused=fused, accumulate=False)
    wl2 = workload.config(2).replace(name="cfg2-no-acc", L=2, prompts=4)
    _full_compare(wl2, lpc=1, k_units=32, export_every=50, device_gen=True, fused=fused, accumulate=False)


@FUSED
@pytest.mark.parametrize("mult", [0.37, 2.5])
def test_caller_supplied_softmax_scale(mult, fused):
    # softmax_scale in the config instead of 1/sqrt(d): a flatter and a sharper softmax, both dtypes and head dims
    for dtype, d in (("bf16", 128), ("f32", 64)):
        wl = workload.Workload("scale-%s-%d" % (dtype, d), L=2, prompts=1, H=6, d=d, dtype=dtype, n0=9, grid_h=7, grid_w=9, W=13,
                               M=10, S=1, R=2, C=7, cadence=5, seed=93, plain=True, softmax_scale=mult / np.sqrt(d))
        _full_compare(wl, fused=fused)
    wl2 = workload.config(2).replace(name="cfg2-scale", L=2, prompts=4, softmax_scale=mult / np.sqrt(128))
    _full_compare(wl2, lpc=1, k_units=32, export_every=50, device_gen=True, fused=fused)


def test_fused_step_against_the_three_calls():
    """The fused step folds the new token into the softmax from registers, as the last row of the first lane
    group, while ssd_decode_attn meets it at its slot in the cache; so the two paths add the same terms in a
    different order and agree to fp32 rounding, not bit for bit.  Positions must be identical at every step
    (inputs whose cuts have a margin), outputs within one rounding of the output dtype, scores within 1e-5."""
    for dtype, d in (("bf16", 128), ("f32", 64)):
        wl = workload.Workload("fused-vs-calls-%s" % dtype, L=2, prompts=2, H=6, d=d, dtype=dtype, n0=9, grid_h=7, grid_w=9,
                               W=13, M=10, S=2, R=2, C=7, cadence=5, seed=97, plain=True)
        ht = workload.head_map(wl)
        data = _to_cuda(workload.generate(wl, head_type=ht))
        sched = workload.compress_schedule(wl)
        units = sample_units(wl, ht, 10 ** 9)
        steps = list(range(wl.n_total))
        o1, e1, _ = gpu_decode(wl, data, ht, sched, units, export_steps=steps, fused=False)
        o2, e2, _ = gpu_decode(wl, data, ht, sched, units, export_steps=steps, fused=True, shadow=False)
        tol = 2.0 ** -7 if dtype == "bf16" else 2e-6                 # relative: one bf16 ulp / a few fp32 ulps
        assert (np.abs(o1 - o2) <= tol * np.maximum(np.abs(o1), 1.0)).all(), float(np.abs(o1 - o2).max())
        for p in steps:
            (p1, s1), (p2, s2) = e1[p]["post"], e2[p]["post"]
            # same tokens retained by every head (slot order is free: compare position -> score)
            for idx in np.ndindex(p1.shape[:3]):
                a = {int(x): float(y) for x, y in zip(p1[idx], s1[idx]) if x >= 0}
                b = {int(x): float(y) for x, y in zip(p2[idx], s2[idx]) if x >= 0}
                assert sorted(a) == sorted(b), ("positions", p, idx)
                assert all(abs(a[k] - b[k]) <= 1e-5 * max(1.0, abs(a[k])) for k in a), ("scores", p, idx)


@FUSED
def test_window_and_budget_per_layer(fused):
    # layer-wise allocation: every layer its own W and M (units of different size, separate launches), also
    # two neighbouring layers that share both (one launch) and a budget larger than the sequence
    wl = workload.Workload("per-layer", L=5, prompts=1, H=6, d=128, dtype="bf16", n0=7, grid_h=6, grid_w=10, W=99, M=99,
                           S=1, R=1, C=4, cadence=3, seed=23, plain=True,
                           W_layers=(24, 5, 5, 1, 13), M_layers=(20, 9, 9, 3, 200))
    _full_compare(wl, fused=fused)
    _full_compare(wl.replace(name="per-layer-calls"), lpc=1, fused=fused)
    wl2 = workload.config(2).replace(name="cfg2-pyramid", L=4, prompts=4, W_layers=(64, 48, 32, 16), M_layers=(96, 64, 32, 16))
    _full_compare(wl2, k_units=32, export_every=50, device_gen=True, fused=fused)


@FUSED
def test_window_and_budget_per_head(fused):
    # head-wise allocation: every head its own W_h or M_h inside units sized for the layer's largest; includes
    # W_h = 1, M_h = 1, a budget larger than the sequence, two equal neighbours, and Algorithm 2's row buffer
    hb = ((24, 5, 1, 7, 200, 3), (9, 9, 30, 2, 1, 17), (13, 40, 6, 6, 11, 1))
    wl = workload.Workload("per-head", L=3, prompts=1, H=6, d=128, dtype="bf16", n0=7, grid_h=6, grid_w=10, W=99, M=99,
                           S=1, R=1, C=4, cadence=3, seed=29, plain=True, head_budget=hb)
    _full_compare(wl, fused=fused)
    _full_compare(wl.replace(name="per-head-calls"), lpc=1, fused=fused)
    _full_compare(wl.replace(name="per-head-alg2", alg2=True, R=0, C=5, cadence=5), fused=fused)
    _full_compare(wl.replace(name="per-head-f32-d64", dtype="f32", d=64, S=2, R=2, C=9, cadence=6), fused=fused)
    # layers whose heads agree (handled like per-layer budgets, two of them sharing a launch) around one whose heads differ
    mixed = ((7, 7, 7, 5, 5, 5), (5, 5, 5, 7, 7, 7), (9, 4, 7, 5, 2, 5), (5, 5, 5, 7, 7, 7))   # W = 7, M = 5 where uniform
    _full_compare(wl.replace(name="per-head-mixed-layers", L=4, spatial_frac=0.5, head_budget=mixed), fused=fused)
    # long row buffer: many evictions per compression, the general selection path with each head's own M_h
    _full_compare(wl.replace(name="per-head-long-buffer", R=3, C=40, cadence=33), fused=fused)
    r = np.random.default_rng(5)
    wl2 = workload.config(2).replace(name="cfg2-per-head", L=3, prompts=4,
                                     head_budget=tuple(tuple(int(x) for x in r.integers(8, 97, 16)) for _ in range(3)))
    _full_compare(wl2, k_units=48, export_every=50, device_gen=True, fused=fused)


@pytest.mark.parametrize("rope", [ssd.SSD_ROPE_HALF, ssd.SSD_ROPE_INTERLEAVED], ids=["half", "interleaved"])
def test_fused_step_with_rotary_embedding(rope):
    # q and k rotated inside the fused step against the oracle's rotation followed by the ordinary oracle route:
    # all four (dtype, head dim), budgets per head, Algorithm 2, and the 1B shape on sampled units
    for dtype, d in (("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)):
        wl = workload.Workload("rope-%s-%d" % (dtype, d), L=2, prompts=2, H=6, d=d, dtype=dtype, n0=9, grid_h=7, grid_w=9,
                               W=13, M=10, S=2, R=2, C=7, cadence=5, seed=81, plain=True)
        _full_compare(wl, fused=True, rope=rope)
    hb = ((24, 5, 1, 7, 40, 3), (9, 9, 30, 2, 1, 17))
    wl = workload.Workload("rope-per-head", L=2, prompts=1, H=6, d=128, dtype="bf16", n0=7, grid_h=6, grid_w=10, W=99, M=99,
                           S=1, R=1, C=4, cadence=3, seed=31, plain=True, head_budget=hb)
    _full_compare(wl, fused=True, rope=rope)
    _full_compare(wl.replace(name="rope-alg2", head_budget=None, W=9, M=7, alg2=True, R=0, C=5, cadence=5), lpc=1, fused=True, rope=rope)
    wl2 = workload.config(2).replace(name="cfg2-rope", L=2, prompts=4)
    _full_compare(wl2, lpc=1, k_units=32, export_every=50, device_gen=True, fused=True, rope=rope)
    # the rotary step dealt to two and three streams: against the oracle, and bit-equal to the one-stream rotary step
    _full_compare(wl2.replace(name="cfg2-rope-split"), lpc=1, k_units=32, export_every=50, device_gen=True, fused=True, rope=rope, split=2)
    wl3 = workload.Workload("rope-split3", L=2, prompts=5, H=6, d=64, dtype="bf16", n0=7, grid_h=6, grid_w=10, W=9, M=7, S=1, R=1, C=4,
                            cadence=3, seed=37, plain=True)
    ht = workload.head_map(wl3)
    data = _to_cuda(workload.generate(wl3, head_type=ht))
    sched = workload.compress_schedule(wl3)
    units = sample_units(wl3, ht, 10 ** 9)
    last = [wl3.n_total - 1]
    o1, e1, _ = gpu_decode(wl3, data, ht, sched, units, export_steps=last, fused=True, rope=rope, shadow=False)
    o2, e2, c2 = gpu_decode(wl3, data, ht, sched, units, export_steps=last, fused=True, rope=rope, shadow=False, split=3)
    assert c2.split_plan(wl3.L, 3) == (4, 3)
    assert np.array_equal(o1, o2)
    for a, b in zip(e1[last[0]]["post"], e2[last[0]]["post"]):
        assert np.array_equal(a, b)
    # parts of 1024 and of 2048 units (four and two waves per unit, each rotating the query for itself)
    wide = workload.Workload("rope-split-parts-of-1024", L=2, prompts=8, H=128, d=64, dtype="bf16", n0=8, grid_h=6, grid_w=6, W=12,
                             M=10, S=1, R=1, C=4, cadence=3, seed=75, plain=True)
    c = _full_compare(wide, lpc=1, k_units=32, export_every=4, device_gen=True, fused=True, rope=rope, split=2)
    assert c.last_launch_shape()[:2] == (4, 14)
    c = _full_compare(wide.replace(name="rope-split-parts-of-2048", prompts=16, d=128, seed=77), lpc=1, k_units=32, export_every=4,
                      device_gen=True, fused=True, rope=rope, split=2)
    assert c.last_launch_shape()[:2] == (4, 12)


def _fma_f32(a, b, c):
    """fma(a, b, c) on float32 arrays, correctly rounded: the product of two float32 values is exact in double,
    the sum is formed in double with its rounding error recovered exactly, and the final rounding to float32 is
    corrected where the rounded double sits exactly half way between two float32 values."""
    a, b, c = (np.asarray(x, np.float32).astype(np.float64) for x in (a, b, c))
    prod = a * b                                  # exact: 24 + 24 significand bits
    s = prod + c
    bb = s - prod
    err = (prod - (s - bb)) + (c - bb)            # s + err = prod + c exactly
    r = s.astype(np.float32)
    up = np.nextafter(r, np.float32(np.inf)).astype(np.float64)
    dn = np.nextafter(r, np.float32(-np.inf)).astype(np.float64)
    r64 = r.astype(np.float64)
    tie_up = (s == (r64 + up) / 2) & (err > 0)    # the double sat on a tie that the exact value is above
    tie_dn = (s == (r64 + dn) / 2) & (err < 0)
    r = np.where(tie_up, up.astype(np.float32), r)
    r = np.where(tie_dn, dn.astype(np.float32), r)
    return r.astype(np.float32)


def _rotate_rows_float_form(wl, x, rope):
    """The arithmetic the header of ssd_decode_step_rope states for the rotation -- float32, one product and one
    fused multiply-add per element, one rounding to the cache dtype -- written out with numpy, for the
    GPU-against-GPU equivalence below.  (The oracle's rotation is the definition in double; it is what every
    parity test of the rotary step compares with.)"""
    cos_t, sin_t = workload.rope_tables(wl.n_total, wl.d)
    xf = x.to(torch.float32).cpu().numpy()
    n, d = xf.shape[0], wl.d
    out = np.empty_like(xf)
    ia = np.arange(d // 2) if rope == ssd.SSD_ROPE_HALF else 2 * np.arange(d // 2)
    ib = ia + d // 2 if rope == ssd.SSD_ROPE_HALF else ia + 1
    shape = (n,) + (1,) * (xf.ndim - 2) + (d // 2,)
    c, sn = cos_t.reshape(shape), sin_t.reshape(shape)
    a, b = xf[..., ia], xf[..., ib]
    ta, tb = (b * sn).astype(np.float32), (a * sn).astype(np.float32)
    out[..., ia] = _fma_f32(a, np.broadcast_to(c, a.shape), -ta)
    out[..., ib] = _fma_f32(b, np.broadcast_to(c, b.shape), tb)
    return torch.from_numpy(out).to(wl.torch_dtype)


def test_rotary_step_equals_plain_step_on_rotated_rows():
    # the stated equivalence, bit for bit, GPU against GPU: rotating and rounding q and k beforehand with the
    # arithmetic the header states and calling the plain step gives the same outputs and the same cache
    wl = workload.Workload("rope-equiv", L=2, prompts=2, H=8, d=128, dtype="bf16", n0=5, grid_h=6, grid_w=8, W=11, M=9,
                           S=1, R=1, C=3, cadence=2, seed=83, plain=True)
    ht = workload.head_map(wl)
    data = _to_cuda(workload.generate(wl, head_type=ht))
    sched = workload.compress_schedule(wl)
    units = sample_units(wl, ht, 10 ** 9)
    for rope in (ssd.SSD_ROPE_HALF, ssd.SSD_ROPE_INTERLEAVED):
        o1, e1, _ = gpu_decode(wl, data, ht, sched, units, export_steps=[wl.n_total - 1], fused=True, rope=rope, shadow=False)
        rot = dict(data)
        rot["q"] = _rotate_rows_float_form(wl, data["q"], rope).cuda()
        rot["k"] = _rotate_rows_float_form(wl, data["k"], rope).cuda()
        o2, e2, _ = gpu_decode(wl, rot, ht, sched, units, export_steps=[wl.n_total - 1], fused=True, shadow=False)
        assert np.array_equal(o1, o2)
        for a, b in zip(e1[wl.n_total - 1]["post"], e2[wl.n_total - 1]["post"]):
            assert np.array_equal(a, b)


@FUSED
def test_algorithm2_spatial_heads_read_the_row_buffer(fused):
    # Algorithm 2 as printed: row buffer of C tokens shared by both head types, emptied at each compression
    # (R = 0), compression when it is full; and a variant that keeps R recent tokens and compresses early
    base = dict(L=2, prompts=1, H=6, d=128, dtype="bf16", n0=5, grid_h=8, grid_w=12, seed=17, plain=True, alg2=True)
    _full_compare(workload.Workload("alg2-literal", W=16, M=12, S=1, R=0, C=12, cadence=12, **base), fused=fused)
    _full_compare(workload.Workload("alg2-recent", W=9, M=7, S=2, R=3, C=10, cadence=5, **base), fused=fused)
    _full_compare(workload.Workload("alg2-all-spatial", W=6, M=4, S=1, R=0, C=4, cadence=4, **base),
                  ht=np.zeros((2, 6), np.uint8), fused=fused)
    wl = workload.config(2).replace(name="cfg2-alg2", L=2, prompts=4, alg2=True, R=0, C=24, cadence=24)
    _full_compare(wl, k_units=32, export_every=50, device_gen=True, fused=fused)


@FUSED
def test_maximum_sizes(fused):
    # 128 heads (both words of the head mask, the type lists reversed in the odd layer)
    wl = workload.Workload("H128", L=2, prompts=1, H=128, d=64, dtype="bf16", n0=3, grid_h=5, grid_w=6, W=7, M=5, S=1, R=1,
                           C=3, cadence=2, spatial_frac=0.5, seed=41, plain=True)
    _full_compare(wl, k_units=96, fused=fused)
    _full_compare(wl.replace(name="H128-uneven", spatial_frac=0.25), k_units=96, lpc=1, fused=fused)
    r = np.random.default_rng(7)
    _full_compare(wl.replace(name="H128-per-head", head_budget=tuple(tuple(int(x) for x in r.integers(1, 12, 128)) for _ in range(2))),
                  k_units=96, fused=fused)
    # the largest batch the config accepts (65534 sequences: the grid's y extent), sampled units
    wl = workload.Workload("B65534", L=1, prompts=32767, H=2, d=64, dtype="bf16", n0=2, grid_h=3, grid_w=4, W=3, M=2, S=1, R=1,
                           C=2, cadence=1, spatial_frac=0.5, seed=45, plain=True)
    _full_compare(wl, k_units=64, device_gen=True, fused=fused)
    # the largest window the config accepts (a ring that never wraps here: everything is retained)
    wl = workload.Workload("W65535", L=1, prompts=1, H=2, d=128, dtype="bf16", n0=4, grid_h=6, grid_w=8, W=65535, M=4, S=0,
                           R=1, C=2, cadence=1, spatial_frac=1.0, seed=43, plain=True)
    _full_compare(wl, fused=fused)
    # M + C = 4096, the largest semantic unit: 4096 rows attended per step at the end, a compression that ranks
    # 3904 candidates and evicts 904 of them (stand-alone kernel, a whole workgroup per head), a spatial window
    # of 3500 rows beside it
    wl = workload.Workload("M+C=4096", L=1, prompts=1, H=2, d=64, dtype="bf16", n0=4, grid_h=64, grid_w=64, W=3500, M=3000,
                           S=2, R=96, C=1096, cadence=1000, spatial_frac=0.5, seed=47, plain=True)
    _full_compare(wl, export_every=500, fused=fused)


@FUSED
def test_few_long_units_take_the_shared_unit_launch(fused):
    # the launch the library picks by itself for at most 2048 units of at least 96 rows: four waves per unit
    wl = workload.Workload("few-long", L=2, prompts=2, H=4, d=128, dtype="bf16", n0=6, grid_h=12, grid_w=14, W=100, M=97,
                           S=1, R=2, C=30, cadence=25, seed=53, plain=True)
    _full_compare(wl, fused=fused)
    _full_compare(wl.replace(name="few-long-f32", dtype="f32", d=64, alg2=True, R=0, C=25), lpc=1, fused=fused)


def test_unbounded_window_and_budget_equal_dense_kernel():
    wl = workload.Workload("unbounded", L=1, prompts=1, H=4, d=128, dtype="bf16", n0=5, grid_h=6, grid_w=7, W=64,
                           M=64, S=0, R=1, C=2, cadence=1, seed=11, plain=True)
    ht = workload.head_map(wl)
    data = _to_cuda(workload.generate(wl, head_type=ht))
    units = sample_units(wl, ht, 10 ** 9)
    outs, _, _ = gpu_decode(wl, data, ht, workload.compress_schedule(wl), units, export_steps=[wl.n_total - 1])
    K = workload.dense_layout(data["k"])[0]
    V = workload.dense_layout(data["v"])[0]
    out = torch.empty((wl.B, wl.H, wl.d), dtype=torch.bfloat16, device="cuda")
    for p in range(wl.n_total):
        ssd.ssd_dense_decode_attn(data["q"][p, 0], K, V, out, wl.B, wl.H, wl.d, "bf16", wl.n_total, p + 1)
        dense = out.float().cpu().numpy().reshape(-1, wl.d)
        # both kernels round to bf16 at the end: allow one bf16 ulp of the value
        np.testing.assert_allclose(outs[p], dense, atol=4e-3, rtol=8e-3)


# ------------------------------------------------------------------ paper-shaped, full size ----------

@FUSED
def test_config2_full_size_sampled_units(fused):
    wl = workload.config(2)
    _full_compare(wl, k_units=48, export_every=64, device_gen=True, fused=fused)


@FUSED
def test_config2_per_layer_launches(fused):
    wl = workload.config(2).replace(name="cfg2-perlayer", L=4)
    _full_compare(wl, lpc=1, k_units=24, export_every=96, device_gen=True, fused=fused)


@FUSED
def test_config4_high_resolution_row_buffer(fused):
    wl = workload.config(4)
    _full_compare(wl, k_units=32, export_every=256, device_gen=True, fused=fused)


def test_config3_headline_shape_per_layer_fused_sampled_units():
    # the configuration and launch shape bench.py times: 7B-shaped, one fused launch per layer
    wl = workload.config(3)
    _full_compare(wl, lpc=1, k_units=64, export_every=128, device_gen=True, fused=True)


@pytest.mark.parametrize("ch,wpu", [(1, 1), (2, 1), (4, 1), (1, 2), (2, 2), (4, 2), (1, 4), (2, 4), (4, 4),
                                    (2, 12), (4, 12), (2, 14), (4, 14)])
def test_every_launch_shape_variant(ch, wpu):
    # all kernel variants the tuning knobs can select must give the same results (12, 14: two / four waves share a unit)
    wl = workload.Workload("variant", L=2, prompts=1, H=6, d=128, dtype="bf16", n0=7, grid_h=9, grid_w=10, W=37,
                           M=21, S=2, R=2, C=9, cadence=6, seed=13, plain=True)
    for new_rows in (1, 2):       # the fused step's new rows stored at the start of / after the row stream
        shape = (ch, wpu, new_rows)
        _full_compare(wl, fused=False, shape=shape)
        _full_compare(wl, fused=True, shape=shape)
        if wpu > 4:           # also the other dtype and head dim, a long row buffer (general selection) and Algorithm 2
            _full_compare(wl.replace(name="variant-f32-64", dtype="f32", d=64), fused=True, shape=shape)
            _full_compare(wl.replace(name="variant-long", R=3, C=40, cadence=33), fused=True, shape=shape)
            _full_compare(wl.replace(name="variant-alg2", alg2=True, R=0, C=6, cadence=6), fused=True, shape=shape)
            _full_compare(wl.replace(name="variant-empty-parts", W=3, M=2, S=0, R=1, C=2, cadence=1), fused=True, shape=shape)
            if ch == 4:       # budgets per head and the rotary step exist with four wave-loads per chunk
                hb = ((24, 5, 1, 7, 40, 3), (9, 9, 30, 2, 1, 17))
                heads = wl.replace(name="variant-per-head", W=99, M=99, head_budget=hb)
                _full_compare(heads, fused=False, shape=shape)
                _full_compare(heads, fused=True, shape=shape)
                _full_compare(heads.replace(name="variant-per-head-alg2", alg2=True, R=0, C=6, cadence=6), fused=True, shape=shape)
                for rope in (ssd.SSD_ROPE_HALF, ssd.SSD_ROPE_INTERLEAVED):
                    _full_compare(wl.replace(name="variant-rope"), fused=True, shape=shape, rope=rope)
                    _full_compare(heads.replace(name="variant-per-head-rope"), fused=True, shape=shape, rope=rope)


@pytest.mark.parametrize("fused", [False, True], ids=["three-calls", "fused-step"])
def test_few_long_heads_beside_many_short_ones(fused):
    """The head mix the paper's threshold produces (Sec. 3.3, Table 6: a few semantic heads with a large budget beside many
    spatial heads with a short window), and its mirror image: once one head type streams twice the rows of the other and
    has at most a quarter of the heads, the library gives every unit two waves, or four if the long type is the semantic
    one with at least 96 rows."""
    few_sem = workload.Workload("few-long-semantic", L=2, prompts=3, H=16, d=128, dtype="bf16", n0=12, grid_h=8, grid_w=12, W=8, M=40,
                                S=1, R=1, C=3, cadence=2, seed=111, plain=True, spatial_frac=0.875)
    c = _full_compare(few_sem, lpc=1, k_units=40, export_every=3, fused=fused)
    assert c.last_launch_shape()[:2] == (4, 12)                      # 43 rows against 9
    c = _full_compare(few_sem.replace(name="few-very-long-semantic", M=96, seed=113), lpc=None, k_units=40, export_every=3, fused=fused)
    assert c.last_launch_shape()[:2] == (4, 14)                      # 99 rows against 9
    few_sp = few_sem.replace(name="few-long-spatial", W=70, M=10, spatial_frac=0.125, seed=115, d=64, dtype="f32")
    c = _full_compare(few_sp, lpc=1, k_units=40, export_every=3, fused=fused)
    assert c.last_launch_shape()[:2] == (4, 12)                      # 71 rows against 13
    c = _full_compare(few_sem.replace(name="few-long-semantic-alg2", alg2=True, R=0, C=6, cadence=6, M=60, seed=117), lpc=1, k_units=40,
                      export_every=3, fused=fused)
    assert c.last_launch_shape()[:2] == (4, 12)                      # 60 rows and the row buffer against 9 and the row buffer
    # as many long heads as short ones: the plain shape
    c = _full_compare(few_sem.replace(name="half-long-semantic", spatial_frac=0.5, seed=119), lpc=1, k_units=40, export_every=3, fused=fused)
    assert c.last_launch_shape()[1] in (1, 4)
    if fused:       # the same mix through the rotary step and through the split call
        c = _full_compare(few_sem.replace(name="few-long-semantic-rope", seed=123), lpc=1, k_units=40, export_every=3, fused=True,
                          rope=ssd.SSD_ROPE_HALF)
        assert c.last_launch_shape()[:2] == (4, 12)
        c = _full_compare(few_sem.replace(name="few-very-long-semantic-split", M=96, prompts=4, seed=125), lpc=1, k_units=40, export_every=3,
                          fused=True, split=2)
        assert c.last_launch_shape()[:2] == (4, 14)


@pytest.mark.parametrize("dtype,d,rows,ch,ch3", [("bf16", 128, 33, 4, 4), ("bf16", 128, 64, 4, 5), ("bf16", 128, 65, 5, 5), ("bf16", 128, 80, 5, 4),
                                                 ("bf16", 128, 81, 4, 4), ("bf16", 128, 129, 5, 5), ("bf16", 64, 130, 5, 5),
                                                 ("f32", 64, 66, 5, 5), ("f32", 128, 33, 5, 5)])
def test_small_calls_give_a_unit_four_waves_and_one_chunk_if_it_fits(dtype, d, rows, ch, ch3):
    """Small calls: four waves per unit, and five loads per chunk where that saves a chunk; one chunk holds 4 * ch loads of 1 KB.  `rows`: what the units stream beside the new token; the three calls stream the new one as well (ch3)."""
    base = workload.Workload("small-call-%d" % rows, L=2, prompts=2, H=6, d=d, dtype=dtype, n0=9, grid_h=4, grid_w=rows // 2, W=rows,
                             M=rows - 1, S=1, R=1, C=3, cadence=1, seed=300 + rows, plain=True)
    for fused in (False, True):
        c = _full_compare(base, lpc=1, k_units=12, export_every=5, fused=fused)
        assert c.last_launch_shape()[:2] == (ch if fused else ch3, 14), c.last_launch_shape()
    c = _full_compare(base.replace(name=base.name + "-rope"), lpc=None, k_units=12, export_every=7, fused=True, rope=ssd.SSD_ROPE_HALF)
    assert c.last_launch_shape()[:2] == (ch, 14)
    hb = np.random.default_rng(rows).integers(rows - 12, rows, (2, 6))
    hb[:, 0] = rows                                               # the longest head of each type decides
    hb[:, 5] = rows
    c = _full_compare(base.replace(name=base.name + "-heads", W=rows, M=rows, head_budget=hb.tolist()), lpc=1, k_units=12, export_every=7,
                      fused=True)
    assert c.last_launch_shape()[1] == 14


@pytest.mark.parametrize("rope,heads", [(0, False), (1, False), (0, True), (1, True)])
def test_a_reported_launch_shape_pins_the_same_results(rope, heads):
    """What ssd_cache_last_launch_shape reports, handed to ssd_cache_set_launch_shape, gives the same launch: every bit equal."""
    wl = workload.Workload("pinned", L=1, prompts=2, H=6, d=128, dtype="bf16", n0=9, grid_h=4, grid_w=33, W=66, M=66, S=1, R=1, C=3, cadence=1,
                           seed=21, plain=True, head_budget=[[66, 40, 50, 33, 45, 66]] if heads else None)
    ht = workload.head_map(wl)
    data = workload.generate(wl, device="cuda", head_type=ht)
    sched, units, last = workload.compress_schedule(wl), sample_units(wl, ht, 10 ** 9), [wl.n_total - 1]
    a, b = (make_cache(wl, ht, torch.device("cuda")) for _ in range(2))
    for c in (a, b):
        gpu_decode(wl, data, ht, sched, units, p_end=last[0], fused=True, rope=rope, cache=c, shadow=False)
    o1, e1, _ = gpu_decode(wl, data, ht, sched, units, export_steps=last, p_begin=last[0], fused=True, rope=rope, cache=a, shadow=False)
    shape = a.last_launch_shape()
    assert shape[:2] == (5, 14)
    o2, e2, _ = gpu_decode(wl, data, ht, sched, units, export_steps=last, p_begin=last[0], fused=True, rope=rope, cache=b, shape=shape, shadow=False)
    assert b.last_launch_shape() == shape
    assert np.array_equal(o1, o2)
    assert all(np.array_equal(x, y) for x, y in zip(e1[last[0]]["post"], e2[last[0]]["post"]))


@pytest.mark.parametrize("dtype,d,rows,prompts,rope,shape", [
    ("bf16", 128, 40, 32, 0, (4, 14)), ("bf16", 128, 40, 33, 0, (4, 1)),                       # 512 units and 528
    ("bf16", 128, 65, 48, 0, (5, 14)), ("bf16", 128, 65, 48, 1, (4, 1)), ("bf16", 128, 65, 49, 0, (4, 1)),    # 768 in one chunk, 784
    ("bf16", 128, 81, 48, 0, (4, 1)), ("bf16", 128, 100, 48, 1, (4, 14)), ("bf16", 128, 129, 48, 0, (5, 14)),
    ("f32", 128, 33, 40, 0, (5, 14)), ("f32", 128, 41, 40, 0, (4, 1)), ("bf16", 64, 70, 36, 0, (4, 1)),
    ("bf16", 128, 257, 2, 0, (4, 14)), ("bf16", 128, 273, 2, 0, (5, 14))])                    # three and two loads of the last chunk unused
def test_calls_around_512_and_768_units(dtype, d, rows, prompts, rope, shape):
    """Which launch a call of 16 units per prompt takes, and its results."""
    wl = workload.Workload("call-of-%d-units" % (16 * prompts), L=1, prompts=prompts, H=8, d=d, dtype=dtype, n0=9, grid_h=4, grid_w=rows // 2, W=rows,
                           M=rows - 1, S=1, R=1, C=3, cadence=1, seed=500 + rows, plain=True)
    c = _full_compare(wl, lpc=1, k_units=8, export_every=23, device_gen=True, fused=True, rope=rope)
    assert c.last_launch_shape()[:2] == shape


@pytest.mark.parametrize("fused", [False, True], ids=["three-calls", "fused-step"])
def test_selection_with_few_evictions_among_many_candidates(fused):
    """More than 128 candidates and one to a few evictions per compression: the step kernel's wave takes the smallest keys
    out one by one instead of ranking all candidates.  The kept sets must be the oracle's at every cut (exported every
    step once the budget is full), with one, two, three and five evictions per cut and 131 to 310 candidates."""
    for M, cadence, C, R in ((130, 1, 2, 1), (150, 2, 4, 1), (200, 3, 6, 2), (300, 5, 7, 1)):
        wl = workload.Workload("few-evictions-M%d-c%d" % (M, cadence), L=1, prompts=1, H=4, d=64, dtype="f32", n0=M + 10, grid_h=4,
                               grid_w=6, W=5, M=M, S=1, R=R, C=C, cadence=cadence, seed=121 + M, plain=True, spatial_frac=0.25)
        _full_compare(wl, fused=fused, export_every=1)


@pytest.mark.parametrize("dtype,d,M,R,heads", [("f32", 64, 126, 1, False), ("bf16", 128, 127, 1, False), ("f32", 64, 128, 1, False), ("bf16", 128, 128, 0, False),
                                               ("f32", 128, 129, 2, False), ("bf16", 64, 191, 1, False), ("f32", 64, 192, 0, False),
                                               ("bf16", 128, 321, 1, False), ("f32", 64, 200, 1, True), ("bf16", 128, 128, 0, True)])
def test_one_eviction_among_any_number_of_candidates(dtype, d, M, R, heads):
    """Compression after every token evicts one of M + 1, settled in registers however many there are: around 64, 128, 192 and
    320 candidates, with the new token among them (R = 0) and not, and with heads of fewer than M."""
    own = [[5, M, max(1, M - 70), M // 2], [5, M // 2, M, M - 1]] if heads else None
    wl = workload.Workload("one-eviction-M%d-R%d" % (M, R), L=2, prompts=1, H=4, d=d, dtype=dtype, n0=M - 6, grid_h=4, grid_w=6, W=5 if not heads else M,
                           M=M, S=1, R=R, C=R + 1, cadence=1, seed=700 + M, plain=True, spatial_frac=0.25, head_budget=own)
    _full_compare(wl, fused=True, lpc=1, export_every=1)


@pytest.mark.parametrize("shape,dtype,d,R,rope,lpc,heads", [((4, 1, 0), "f32", 64, 1, 0, 1, False), ((4, 2, 0), "bf16", 128, 1, 0, None, False), ((4, 4, 0), "f32", 128, 0, 1, None, False),
                                                            ((4, 4, 0), "bf16", 128, 1, 2, 1, False), ((4, 12, 0), "bf16", 64, 1, 0, None, False), ((4, 14, 0), "f32", 64, 1, 1, None, False),
                                                            ((5, 14, 0), "bf16", 128, 1, 0, 1, False), ((2, 4, 0), "f32", 64, 1, 0, None, False), ((4, 4, 0), "f32", 64, 1, 0, 1, True),
                                                            ((4, 12, 0), "f32", 64, 1, 1, 1, True)])
def test_one_eviction_among_many_candidates_in_every_launch_shape(shape, dtype, d, R, rope, lpc, heads):
    """More than 128 candidates: one wave per unit and units shared, the rotary step, budgets per head (some heads with fewer), one layer per
    call and all; two wave-loads per chunk rank through LDS."""
    own = [[5, 140, 70, 128], [5, 127, 140, 129]] if heads else None
    wl = workload.Workload("one-eviction-shape", L=2, prompts=1, H=4, d=d, dtype=dtype, n0=134, grid_h=4, grid_w=4, W=5 if not heads else 140, M=140, S=1,
                           R=R, C=R + 1, cadence=1, seed=91, plain=True, spatial_frac=0.25, head_budget=own)
    _full_compare(wl, fused=True, lpc=lpc, export_every=1, rope=rope, shape=shape)


@pytest.mark.parametrize("prompts,H,frac,rows,lpc", [(8, 16, 0.5, 9, 1), (9, 16, 0.5, 40, 1), (19, 32, 0.25, 33, 1), (19, 16, 0.5, 20, None), (7, 16, 0.5, 9, 1),
                                                     (43, 64, 0.5, 9, 1), (66, 32, 0.75, 12, None)])
def test_units_dealt_to_the_xcds(prompts, H, frac, rows, lpc):
    """A multiple of eight workgroups per sequence and head type: whole blocks of 16 sequences are dealt two at a time, the rest and
    fewer as they come; one and four units per workgroup, one layer and several per call."""
    wl = workload.Workload("dealt-%d-%d" % (prompts, H), L=2, prompts=prompts, H=H, d=128, dtype="bf16", n0=rows, grid_h=2, grid_w=5, W=rows, M=rows - 1,
                           S=1, R=1, C=2, cadence=1, seed=900 + prompts, plain=True, spatial_frac=frac)
    for fused in (False, True):
        _full_compare(wl, lpc=lpc, k_units=48, export_every=4, device_gen=True, fused=fused)


def test_determinism_same_inputs_same_bits():
    wl = workload.config(2).replace(name="cfg2-determinism", L=2, prompts=4, grid_h=6)
    ht = workload.head_map(wl)
    data = workload.generate(wl, device="cuda", head_type=ht)
    units = sample_units(wl, ht, 10 ** 9)
    sched = workload.compress_schedule(wl)
    a, ea, _ = gpu_decode(wl, data, ht, sched, units, export_steps=[wl.n_total - 1])
    b, eb, _ = gpu_decode(wl, data, ht, sched, units, export_steps=[wl.n_total - 1])
    np.testing.assert_array_equal(a, b)
    for k in (0, 1):
        np.testing.assert_array_equal(ea[wl.n_total - 1]["post"][k], eb[wl.n_total - 1]["post"][k])


@pytest.mark.parametrize("n_streams", [2, 3, 4])
def test_split_step_on_several_streams_equals_the_one_stream_step(n_streams):
    """ssd_decode_step_split (the schedule bench.py times): the batch dealt to n streams, forked at a token's first
    layer and joined at its last.  Sequences are independent, so with the launch shape pinned outputs and final
    tables must equal the one-stream ssd_decode_step bit for bit, and with the library's own shapes too wherever the
    two calls give a unit the same number of waves (here: every part has at most 512 units); larger parts may take
    several waves per unit, which changes the order of the fp32 sums: there the two calls agree to rounding.  Includes a batch that does not divide evenly (10 sequences
    on 3 and 4 streams), a long row buffer whose selection runs in the stand-alone kernel, budgets per head and
    Algorithm 2."""
    cases = [workload.config(2).replace(name="cfg2-split", L=3, prompts=8, grid_h=5),
             workload.config(2).replace(name="cfg2-split-uneven", L=2, prompts=5, grid_h=4),
             workload.Workload("split-long-buffer", L=2, prompts=3, H=4, d=64, dtype="f32", n0=6, grid_h=40, grid_w=40, W=30,
                               M=900, S=1, R=4, C=400, cadence=390, seed=61, plain=True),
             # 40 sequences x 128 heads x 3 layers per call: more parts than streams (4 parts of 10 sequences on 2 streams)
             workload.Workload("split-many-parts", L=3, prompts=20, H=128, d=64, dtype="bf16", n0=3, grid_h=4, grid_w=5, W=7, M=5,
                               S=1, R=1, C=3, cadence=2, seed=67, plain=True),
             workload.Workload("split-per-head-alg2", L=2, prompts=3, H=6, d=128, dtype="bf16", n0=7, grid_h=6, grid_w=10, W=99,
                               M=99, S=1, R=0, C=5, cadence=5, seed=63, plain=True, alg2=True,
                               head_budget=((24, 5, 1, 7, 40, 3), (9, 9, 30, 2, 1, 17)))]
    for wl in cases:
        say("split case", wl.name, "B", wl.B, "streams", n_streams)
        if wl.name == "split-many-parts" and n_streams == 2:
            assert make_cache(wl, workload.head_map(wl)).split_plan(wl.L, 2) == (10, 4)
        ht = workload.head_map(wl)
        data = workload.generate(wl, device="cuda", head_type=ht)
        sched = workload.compress_schedule(wl)
        units = sample_units(wl, ht, 10 ** 9)
        last = [wl.n_total - 1]
        for lpc in (1, None):
            span = wl.L if lpc is None else lpc
            for shape in ((4, 1, 0), None):
                o1, e1, c1 = gpu_decode(wl, data, ht, sched, units, layers_per_call=lpc, export_steps=last, fused=True, shadow=False,
                                        shape=shape)
                o2, e2, c2 = gpu_decode(wl, data, ht, sched, units, layers_per_call=lpc, export_steps=last, fused=True, shadow=False,
                                        shape=shape, split=n_streams)
                part_units = c2.split_plan(span, n_streams)[0] * wl.H * span
                waves = lambda c: (c.last_launch_shape()[0], max(1, c.last_launch_shape()[1] - 10))     # loads per chunk, waves per unit
                exact = shape is not None or part_units <= 512
                assert not exact or waves(c1) == waves(c2), (wl.name, c1.last_launch_shape(), c2.last_launch_shape())
                if shape is None and 512 < part_units <= 2048:
                    # the shapes ssd_decode_step_split takes for parts of these sizes: two or four waves per unit
                    assert c2.last_launch_shape()[:2] == ((4, 12) if part_units > 1024 else (4, 14)), (wl.name, c2.last_launch_shape())
                    assert c1.last_launch_shape()[1] in (1, 4)
                    say("   parts of", part_units, "units take shape", c2.last_launch_shape(), "- compared to rounding")
                if exact:
                    assert np.array_equal(o1, o2), ("outputs differ", wl.name, lpc, shape)
                else:
                    check_outputs(o2, o1, wl.dtype, "split against one stream, %s" % wl.name)
                for a, b in zip(e1[last[0]]["post"], e2[last[0]]["post"]):
                    if exact or a.dtype.kind == "i":
                        assert np.array_equal(a, b), ("tables differ", wl.name, lpc, shape)
                    else:
                        np.testing.assert_allclose(b, a, rtol=1e-5, atol=1e-6)


def test_split_step_against_the_oracle():
    # the split schedule through the ordinary oracle comparison, own-score checks included
    wl = workload.config(2).replace(name="cfg2-split-oracle", L=2, prompts=6)
    _full_compare(wl, lpc=1, k_units=32, export_every=50, device_gen=True, fused=True, split=2)
    _full_compare(wl.replace(name="cfg2-split3-oracle"), lpc=1, k_units=32, export_every=50, device_gen=True, fused=True, split=3)
    # parts of 1024 and of 2048 units: the sizes at which a part of a split call takes four and two waves per unit
    wide = workload.Workload("split-parts-of-1024", L=2, prompts=8, H=128, d=64, dtype="bf16", n0=8, grid_h=6, grid_w=6, W=12, M=10,
                             S=1, R=1, C=4, cadence=3, seed=71, plain=True)
    c = _full_compare(wide, lpc=1, k_units=48, export_every=4, device_gen=True, fused=True, split=2)
    assert c.last_launch_shape()[:2] == (4, 14)
    c = _full_compare(wide.replace(name="split-parts-of-2048", prompts=16, seed=73), lpc=1, k_units=48, export_every=4, device_gen=True,
                      fused=True, split=2)
    assert c.last_launch_shape()[:2] == (4, 12)
    # parts that fall on two sides of a shape boundary: 10 sequences x 64 heads (four waves per unit) and 8 x 64 (one)
    c = _full_compare(wide.replace(name="split-parts-of-640-and-512", prompts=9, H=64, seed=85), lpc=1, k_units=48, export_every=4,
                      device_gen=True, fused=True, split=2)
    assert c.split_plan(1, 2) == (10, 2) and c.last_launch_shape()[:2] == (4, 1)
    # the same part sizes with a window / budget per head (128 heads, seeded budgets of 3 to 20 rows)
    hb = np.random.default_rng(79).integers(3, 21, (2, 128)).tolist()
    heads = wide.replace(name="split-per-head-parts-of-1024", W=20, M=20, head_budget=hb, seed=81)
    c = _full_compare(heads, lpc=1, k_units=48, export_every=4, device_gen=True, fused=True, split=2)
    assert c.last_launch_shape()[:2] == (4, 14)
    c = _full_compare(heads.replace(name="split-per-head-parts-of-2048", prompts=16, seed=83), lpc=1, k_units=48, export_every=4,
                      device_gen=True, fused=True, split=2)
    assert c.last_launch_shape()[:2] == (4, 12)


def test_config3_headline_shape_split_on_two_streams_sampled_units():
    # the configuration and schedule of bench.py's headline: 7B-shaped, one fused call per layer, two streams
    wl = workload.config(3)
    _full_compare(wl, lpc=1, k_units=64, export_every=128, device_gen=True, fused=True, split=2)


def test_config3_launch_shape_plain_inputs_sampled_units():
    # the headline's launch shape on inputs without planted structure: every retained row carries weight, so a
    # wrong row anywhere shows in the output.  Four layers keep the oracle's share short; a per-layer launch has the
    # full configuration's shape whatever the layer count.
    wl = workload.config(3).replace(name="cfg3-plain", L=4, plain=True)
    _full_compare(wl, lpc=1, k_units=64, export_every=128, device_gen=True, fused=True)
    _full_compare(wl.replace(name="cfg3-plain-split"), lpc=1, k_units=64, export_every=128, device_gen=True, fused=True, split=2)


@pytest.mark.parametrize("frac,W,M,split", [(0.25, 32, 128, 0), (0.5, 64, 64, 2), (0.75, 128, 32, 2)])
def test_config5_large_batch_online_classification_then_decode(frac, W, M, split):
    """Large-batch shape (B = 512, 32 heads) with the head types found online: a dense profiling run on a
    16-sequence sub-batch feeds ssd_classify_heads, the resulting table drives the compressed decode of the
    whole batch.  Two layers keep the test short; a per-layer launch has the full configuration's shape."""
    import oracle as orc
    wl = workload.config(5).replace(name="cfg5-%d-%d-%d" % (int(frac * 100), W, M), L=2, spatial_frac=frac, W=W, M=M)
    planted = workload.head_map(wl)
    say("case", wl.name, "B", wl.B)
    data = workload.generate(wl, device="cuda", head_type=planted)
    P, T, w = 16, wl.N, wl.w_metric
    far = torch.zeros((wl.L, P, wl.H, T), device="cuda")
    tot = torch.zeros_like(far)
    outd = torch.empty((P, wl.H, wl.d), dtype=wl.torch_dtype, device="cuda")
    ws = torch.empty(ssd.ssd_dense_workspace_bytes(P, wl.H, wl.d, wl.n_total), dtype=torch.uint8, device="cuda")
    sub = {x: data[x][:, :, :P].contiguous() for x in "qkv"}
    Kd = workload.dense_layout(sub["k"])
    Vd = workload.dense_layout(sub["v"])
    for t in range(1, T + 1):
        n = wl.n0 + t
        for l in range(wl.L):
            ssd.ssd_dense_decode_attn(sub["q"][n - 1, l], Kd[l], Vd[l], outd, P, wl.H, wl.d, wl.dtype, wl.n_total, n, 0.0,
                                      far[l, :, :, t - 1:].data_ptr(), tot[l, :, :, t - 1:].data_ptr(), T, wl.n0, w, ws)
    s_gpu = torch.zeros((wl.L, wl.H), device="cuda")
    ty_gpu = torch.zeros((wl.L, wl.H), dtype=torch.uint8, device="cuda")
    ssd.ssd_classify_heads(far, tot, wl.L, P, wl.H, T, 0.5, s_gpu, ty_gpu)
    torch.cuda.synchronize()
    ht = ty_gpu.cpu().numpy()
    np.testing.assert_array_equal(ht, planted)
    far_h, tot_h = far.cpu().numpy(), tot.cpu().numpy()
    s_ref, ty_ref = orc.classify(far_h, tot_h, 0.5)                 # the oracle's reduction on the same masses
    np.testing.assert_array_equal(ty_ref, ht)
    np.testing.assert_allclose(s_gpu.cpu().numpy(), s_ref, atol=1e-5, rtol=1e-4)
    assert (np.abs(s_ref - 0.5) > 0.1).all()
    r = np.random.default_rng(5)
    for _ in range(12):                                             # the masses themselves, on sampled units
        l, p, h = int(r.integers(wl.L)), int(r.integers(P)), int(r.integers(wl.H))
        q_, K_, V_ = workload.unit_arrays(sub, l, p, h)
        f_o, t_o = orc.profile_unit(q_, K_, V_, wl.n0, T, w, wl.scale)
        np.testing.assert_allclose(far_h[l, p, h], f_o, atol=2e-5, rtol=2e-4)
        np.testing.assert_allclose(tot_h[l, p, h], t_o, atol=2e-5, rtol=2e-4)
    del Kd, Vd, sub
    # compressed decode of the full batch with the classified table, fused per-layer launches
    schedule = workload.compress_schedule(wl)
    units = sample_units(wl, ht, 40, seed=2)
    steps = sorted(set(range(0, wl.n_total, 160)) | {wl.n_total - 1})
    # split = 2: the launch configuration bench.py times on this shape (four parts of 128 sequences on two streams)
    outs, exports, cache = gpu_decode(wl, data, ht, schedule, units, layers_per_call=1, export_steps=steps, fused=True, split=split)
    if split:
        assert cache.split_plan(1, split) == (128, 4)
    layers = sorted(set(l for (l, _, _) in units))
    worst, near_ties, t3 = 0.0, 0, 0
    for ui, unit in enumerate(units):
        l, b, h = unit
        host = {x: data[x][:, l:l + 1, b:b + 1, h:h + 1].cpu() for x in "qkv"}
        o_ref, hl, gl, _ = oracle_unit(wl, host, ht[l:l + 1, h:h + 1], schedule, (0, 0, 0))
        li = layers.index(l)
        div = compare_unit_sets(wl, ht, unit, li, exports, hl, gl, schedule)
        upto = wl.n_total if div is None else div[0] + 1
        cut = wl.n_total if div is None else div[0]          # own-score checks up to, not including, a near-tie's step
        t3 += len(check_selection_on_own_scores(wl, ht, unit, li, {p: e for p, e in exports.items() if p < cut}))
        worst = max(worst, check_outputs(outs[:upto, ui], o_ref[:upto], wl.dtype, "unit %s" % (unit,)))
        if div is not None:
            near_ties += 1
            settle_near_tie(wl, data, ht, schedule, unit, li, exports, div[0], True, lpc=1)
    say("  max abs output error %.3e, near-tie units %d of %d, own-score selections checked %d" % (worst, near_ties, len(units), t3))
    assert near_ties <= near_tie_cap(len(units)) and t3 > 0


# SSD_RANDOM_SEEDS=a:b widens the sweep for a one-off run (default: the 64 committed seeds)
_SEEDS = range(*(int(x) for x in os.environ.get("SSD_RANDOM_SEEDS", "0:64").split(":")))


@pytest.mark.parametrize("seed", _SEEDS)
def test_random_small_configurations(seed):
    """Seeded random shapes and policies (both dtypes and head dims, Algorithm 1 and 2, any cadence the row
    buffer allows, budgets per layer or per head, the rotary step or the split step now and then), every unit compared at
    every step, fused and unfused."""
    r = np.random.default_rng(1000 + seed)
    d = int(r.choice([64, 128]))
    dtype = str(r.choice(["bf16", "f32"]))
    L, H = int(r.integers(1, 4)), int(r.integers(1, 9))
    R = int(r.integers(0, 4))
    cadence = int(r.integers(1, 9))
    C_ = R + cadence + int(r.integers(0, 3))
    W, M, S = int(r.integers(1, 40)), int(r.integers(1, 40)), int(r.integers(0, 4))
    alg2 = bool(r.integers(0, 2))
    kw = {}
    if L > 1 and r.random() < 0.4:
        kw = dict(W_layers=tuple(int(x) for x in r.integers(1, 40, L)), M_layers=tuple(int(x) for x in r.integers(1, 40, L)))
    wl = workload.Workload("rand%d" % seed, L=L, prompts=int(r.integers(1, 3)), H=H, d=d, dtype=dtype, n0=int(r.integers(1, 12)),
                           grid_h=int(r.integers(2, 7)), grid_w=int(r.integers(2, 9)), W=W, M=M, S=S, R=R, C=C_, cadence=cadence,
                           spatial_frac=float(r.choice([0.0, 0.25, 0.5, 0.75, 1.0])), seed=int(r.integers(1 << 30)),
                           plain=bool(r.integers(0, 2)), alg2=alg2, **kw)
    lpc = None if r.random() < 0.5 else 1
    if r.random() < 0.35:         # budgets per head instead (drawn last: the other cases keep their draws)
        wl = wl.replace(W_layers=None, M_layers=None, head_budget=tuple(tuple(int(x) for x in r.integers(1, 40, H)) for _ in range(L)))
    rope = int(r.choice([0, 0, ssd.SSD_ROPE_HALF, ssd.SSD_ROPE_INTERLEAVED]))    # the fused leg, now and then with rotary embedding
    split = int(r.choice([0, 0, 2, 3]))                                          # ... and / or dealt to several streams (drawn last)
    _full_compare(wl, lpc=lpc, fused=False)
    _full_compare(wl, lpc=lpc, fused=True, rope=rope, split=split)


@pytest.mark.parametrize("seed", range(12))
def test_random_long_units(seed):
    """Seeded random shapes whose units are few and long enough (at least 96 rows once filled) for the launch in
    which four waves share a unit; every unit compared at every step, fused and unfused."""
    r = np.random.default_rng(5000 + seed)
    d = int(r.choice([64, 128]))
    dtype = str(r.choice(["bf16", "f32"]))
    R = int(r.integers(0, 6))
    cadence = int(r.integers(1, 40))
    C_ = R + cadence + int(r.integers(0, 3))
    wl = workload.Workload("long%d" % seed, L=int(r.integers(1, 3)), prompts=1, H=int(r.integers(1, 5)), d=d, dtype=dtype,
                           n0=int(r.integers(1, 20)), grid_h=int(r.integers(10, 16)), grid_w=int(r.integers(12, 20)),
                           W=int(r.integers(96, 200)), M=int(r.integers(96, 200)), S=int(r.integers(0, 4)), R=R, C=C_, cadence=cadence,
                           spatial_frac=float(r.choice([0.0, 0.5, 1.0])), seed=int(r.integers(1 << 30)), plain=True,
                           alg2=bool(r.integers(0, 2)))
    lpc = None if r.random() < 0.5 else 1
    _full_compare(wl, lpc=lpc, fused=False)
    _full_compare(wl, lpc=lpc, fused=True)
