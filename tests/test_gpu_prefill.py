"""GPU parity of ssd_prefill_scores (accumulated causal attention scores of a prompt, matrix-core kernel)
against the oracle, of the whole prompt pipeline: prefill scores -> dense-source compression -> decode, and of
the classifier-free guidance mix that follows the last layer (ssd_cfg_mix)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_18716_amd as ssd
import workload
from harness import (GAP_MARGIN, check_outputs, compare_unit_sets, gpu_decode, make_cache, near_tie_cap, sample_units, say,
                     settle_near_tie)

pytestmark = pytest.mark.gpu

# scores are sums of up to n probabilities, each from an fp32-accumulated product and the hardware exp2
SCORE_TOL = (2e-4, 2e-4)


def _check_scores(got, ref, what):
    err = np.abs(got - ref)
    bad = err > SCORE_TOL[0] + SCORE_TOL[1] * np.abs(ref)
    assert not bad.any(), "%s: %d of %d scores off (max abs err %.3e)" % (what, int(bad.sum()), bad.size, float(err.max()))


def _case(dtype, d, n, units, seed, scale_mult=1.0, peaky=False):
    say("prefill case", dtype, d, "n", n, "units", units, "seed", seed)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(seed)
    q = torch.randn((units, n, d), generator=g)
    k = torch.randn((units, n, d), generator=g)
    if peaky:      # a few keys that every later query looks at, as a sink token would be
        k[:, :: max(1, n // 3)] *= 3.0
        q += 0.5 * k[:, :1]
    q, k = q.to(tdt), k.to(tdt)
    out = torch.full((units, n), -5.0, device="cuda")
    scale = scale_mult / np.sqrt(d)
    ssd.ssd_prefill_scores(q.cuda(), k.cuda(), units, n, d, dtype, out, 0.0 if scale_mult == 1.0 else scale)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    for u in range(units):
        ref = oracle.prefill_scores(q[u].float().numpy(), k[u].float().numpy(), scale)
        _check_scores(got[u], ref, "unit %d" % u)
    # every query row spreads probability 1 over the keys
    np.testing.assert_allclose(got.sum(axis=1), n, rtol=1e-4)
    return got


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_prefill_scores_match_oracle(dtype, d):
    for i, n in enumerate([1, 2, 31, 32, 33, 64, 100, 129]):     # below, at and across tile edges; ragged tails
        _case(dtype, d, n, 3, 100 + i)
    _case(dtype, d, 257, 2, 7, peaky=True)                        # more query blocks than waves
    _case(dtype, d, 96, 2, 8, scale_mult=2.5, peaky=True)         # caller's scale, sharper softmax


def test_prefill_scores_largest_prompt_and_many_units():
    _case("bf16", 128, 1024, 2, 11, peaky=True)
    _case("bf16", 128, 4096, 1, 13, peaky=True)                   # the longest prompt the entry point takes
    _case("f32", 64, 1500, 1, 14)
    got = _case("bf16", 128, 64, 600, 12)                         # more workgroups than compute units
    assert np.isfinite(got).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("n", [131, 160, 161, 256, 287, 512, 513, 800, 4096])
def test_prefill_scores_long_prompts_at_tile_and_workgroup_edges(dtype, d, n):
    """Above 128 tokens: around whole tiles, around what workgroups hold at a time, in calls of so few units that three workgroups share
    each.  A unit beside the last one must stay as it was.  Tolerance: fp32 sums of up to n terms, each within a few
    roundings of 2^-24 of an argument below 2^5 (4e-6), against 64 bits."""
    say("long prompt", dtype, d, n)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(n)
    q = torch.randn((3, n, d), generator=g)
    k = torch.randn((3, n, d), generator=g)
    k[:, :: 50] *= 2.0                                            # some keys that every later query looks at
    q = (q + 0.3 * k[:, :1]).to(tdt)
    k = k.to(tdt)
    out = torch.full((3, n), -5.0, device="cuda")
    ssd.ssd_prefill_scores(q.cuda(), k.cuda(), 2, n, d, dtype, out)
    torch.cuda.synchronize()
    z = torch.matmul(q.double(), k.double().transpose(1, 2)) / np.sqrt(d)
    ref = torch.softmax(z.masked_fill(torch.ones(n, n, dtype=torch.bool).triu(1), -np.inf), dim=-1).sum(dim=1)
    got = out.cpu().double()
    assert bool((got[2] == -5.0).all())
    err = ((got[:2] - ref[:2]).abs() / ref[:2].clamp_min(1e-3)).max()
    assert float(err) < 1e-5, float(err)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [200, 600])
def test_prefill_scores_long_prompts_take_a_logit_that_is_no_number_as_masked(dtype, n):
    """A key that is no number scores 0 and changes nothing else; a query that is none gives nothing to any key."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(n)
    q, k = (torch.randn((2, n, 64), generator=g).to(tdt) for _ in range(2))
    k[0, 37, 5] = float("nan")
    k[0, n - 1, 5] = float("nan")
    q[0, 150, 3] = float("nan")
    out = torch.empty((2, n), device="cuda")
    ssd.ssd_prefill_scores(q.cuda(), k.cuda(), 2, n, 64, dtype, out)
    z = torch.matmul(q.double(), k.double().transpose(1, 2)) / 8.0
    z = z.masked_fill(torch.isnan(z) | torch.ones(n, n, dtype=torch.bool).triu(1), -np.inf)
    ref = torch.nan_to_num(torch.softmax(z, dim=-1)).sum(dim=1)
    got = out.cpu().double()
    assert float(((got - ref).abs() / ref.clamp_min(1e-3)).max()) < 1e-5
    assert float(got[0, 37]) == 0.0 and float(got[0, n - 1]) == 0.0


def _scores_in_64_bits(q, k):
    n = q.shape[1]
    after = torch.ones((n, n), dtype=torch.bool, device=q.device).triu(1)
    return torch.stack([torch.softmax((a.double() @ b.double().T / np.sqrt(q.shape[2])).masked_fill_(after, -np.inf), dim=-1).sum(dim=0)
                        for a, b in zip(q, k)])


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 129), ("bf16", 64, 385), ("bf16", 128, 513), ("bf16", 128, 769), ("f32", 64, 257), ("f32", 128, 160), ("bf16", 64, 1025)])
@pytest.mark.parametrize("units", [1, 85, 86, 128, 129, 256, 257])
def test_prefill_scores_long_prompts_by_number_of_units(dtype, d, n, units):
    """Where a unit's keys are shared by three, two and one workgroup and where workgroups get smaller; two and three tiles per
    wave.  Tolerance as for the edges above."""
    say("units", dtype, d, n, units)
    g = torch.Generator(device="cuda").manual_seed(n + units)
    q, k = (torch.randn((units, n, d), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
    out = torch.full((units + 1, n), -5.0, device="cuda")
    ssd.ssd_prefill_scores(q, k, units, n, d, dtype, out)
    at = sorted({0, units // 2, units - 1})
    ref = _scores_in_64_bits(q[at], k[at])
    assert bool((out[units] == -5.0).all()) and bool(torch.isfinite(out[:units]).all())
    assert float(((out[at].double() - ref).abs() / ref.clamp_min(1e-3)).max()) < 1e-5
    assert float((out[:units].double().sum(dim=1) / n - 1.0).abs().max()) < 1e-6     # every query gives away a mass of 1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [200, 600, 1100])
@pytest.mark.parametrize("rise", [20.0, 60.0, 200.0, 2000.0])
def test_prefill_scores_long_prompts_whose_logits_rise_late(dtype, n, rise):
    """Keys from 100 on whose logits lie 20 to 2000 above those of all before them, and from 150 on as far below again: more than a
    query's first reference can stand for, and more than fp32 holds at all.  Tolerance: a logit of rise / 2 is a sum of 64 products,
    each partial sum rounded by up to 2^-24 of it, in a probability's numerator as in its denominator."""
    say("rise", dtype, n, rise)
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k = (0.1 * torch.randn((3, n, 64), generator=g, device="cuda") for _ in range(2))
    q[:, :, 0], k[:, :, 0] = 16.0, -0.25 * rise
    k[:, 100:150, 0] = 0.25 * rise
    q, k = (x.to(torch.bfloat16 if dtype == "bf16" else torch.float32) for x in (q, k))
    out = torch.empty((3, n), device="cuda")
    ssd.ssd_prefill_scores(q, k, 3, n, 64, dtype, out)
    ref = _scores_in_64_bits(q, k)
    assert float(((out.double() - ref).abs() / ref.clamp_min(1e-3)).max()) < 64 * 2.0 ** -24 * rise


def _scores_of_given_logits(z, dtype):
    """z [units, n]: the logit (log2 domain) every query of a unit gives key j, exact in fp32.  The kernel's scores and those in 64 bits."""
    units, n = z.shape
    q = torch.zeros((units, n, 64), device="cuda")
    k = torch.zeros((units, n, 64), device="cuda")
    rest = z.clone()
    for i in range(3):                                            # three bf16 pieces hold the 24 bits
        q[:, :, i] = 1.0
        k[:, :, i] = rest.to(torch.bfloat16).float()
        rest = rest - k[:, :, i]
    assert not bool(rest.any())
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    out = torch.empty((units, n), device="cuda")
    ssd.ssd_prefill_scores(q.to(tdt), k.to(tdt), units, n, 64, dtype, out, float(np.log(2.0)))
    after = torch.arange(n, device="cuda")
    ref = torch.empty((units, n), dtype=torch.float64, device="cuda")
    for u in range(units):
        p = torch.where(after[None, :] <= after[:, None], z[u].double()[None, :], torch.tensor(-np.inf, dtype=torch.float64, device="cuda"))
        ref[u] = torch.softmax(p * np.log(2.0), dim=-1).sum(dim=0)
    return out.double(), ref


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("low", [-127.0, -126.25, -130.0, -60.0])
@pytest.mark.parametrize("key", [36, 41, 46, 96])
def test_prefill_scores_long_prompts_two_keys_far_above_all_others(dtype, low, key):
    """Key 0 and one later key, of this or that lane, share every query's mass; all others lie up to 2^130 below.  Tolerance: the probabilities
    are exact halves and the others' sums below 2^-50, so only sums over up to 300 queries are rounded."""
    z = torch.full((2, 300), low, device="cuda")
    z[:, 0] = 0.0
    z[0, key] = 0.0
    got, ref = _scores_of_given_logits(z, dtype)
    say("two keys", dtype, low, key, got[0, [0, key]].tolist())
    assert float(((got - ref).abs() / ref.clamp_min(1e-3)).max()) < 1e-6
    assert float((got.sum(dim=1) / 300 - 1.0).abs().max()) < 1e-6


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [200, 600])
@pytest.mark.parametrize("rise", [12, 19, 24, 60, 90, 99])
def test_prefill_scores_long_prompts_lose_no_precision_to_a_late_rise(dtype, n, rise):
    """From key 100 on logits, each known exactly, spread over one power of two that lies `rise` above the first ones.  A query's sum
    stays below 2^20 or is taken again with a running maximum, so an exponential's argument is below 2^5 and rounded by up to
    2^-20: 3.8e-7 rms of its probability, and as much in the sum it is divided by; with arguments of 60 to 100 it would be 2^-18."""
    g = torch.Generator(device="cuda").manual_seed(n + rise)
    z = torch.floor(torch.rand((3, n), generator=g, device="cuda") * 2.0 ** 23) * 2.0 ** -23
    z[:, :100] = -float(rise)
    got, ref = _scores_of_given_logits(z, dtype)
    heavy = ((got - ref) / ref)[:, 100:n - 10]
    say("late rise", dtype, n, rise, "rms", float(heavy.square().mean().sqrt()), "max", float(heavy.abs().max()))
    assert float(heavy.square().mean().sqrt()) < 6e-7


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 129), ("bf16", 128, 300), ("bf16", 128, 640), ("bf16", 128, 1500), ("bf16", 64, 450), ("f32", 128, 330),
                                       ("f32", 64, 700), ("f32", 128, 4096), ("bf16", 128, 2016), ("bf16", 128, 2017)])
def test_prefill_scores_of_a_unit_do_not_depend_on_the_call(dtype, d, n):
    """A unit's scores are the same to the bit whatever number of units the call has, that is, whether two or three workgroups share
    its keys, and how many waves and tiles a workgroup has; also where references are renewed and where a logit is no number."""
    units = 260 if n < 4000 else 131
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k = (torch.randn((units, n, d), generator=g, device="cuda") for _ in range(2))
    q[1::4, :, 0], k[1::4, :, 0], k[1::4, n // 2:, 0] = 16.0, -6.0, 6.0            # rises half way
    k[2, n // 3, 1] = float("nan")
    q[3, n // 2, 1] = float("nan")
    q, k = (x.to(torch.bfloat16 if dtype == "bf16" else torch.float32) for x in (q, k))
    scores = {}
    for u in (1, 4, 86, 129, 130, units):
        say("units", u, dtype, d, n)
        scores[u] = torch.empty((u, n), device="cuda")
        ssd.ssd_prefill_scores(q, k, u, n, d, dtype, scores[u])
    for u, sc in scores.items():
        assert bool(torch.isfinite(sc).all())
        assert torch.equal(sc, scores[units][:u]), (u, float((sc - scores[units][:u]).abs().max()))
    second = torch.empty((units // 2, n), device="cuda")
    ssd.ssd_prefill_scores(q[units - units // 2:], k[units - units // 2:], units // 2, n, d, dtype, second)
    assert torch.equal(second, scores[units][units - units // 2:])


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 200), ("bf16", 128, 400), ("bf16", 128, 800), ("bf16", 64, 400), ("bf16", 64, 600), ("bf16", 128, 1100),
                                       ("f32", 128, 300), ("f32", 64, 600)])
@pytest.mark.parametrize("units", [3, 129, 257, 600])
def test_prefill_scores_long_prompts_disturbed_units_of_any_call(dtype, d, n, units):
    """Logits that are no numbers and logits that rise late in one unit each, in calls whose workgroups share a unit's keys or not and have
    eight or four waves, with one group of held tiles and with several.  Tolerances as for the tests of each."""
    say("disturbed", dtype, d, n, units)
    g = torch.Generator(device="cuda").manual_seed(n + units)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k = (torch.randn((units, n, d), generator=g, device="cuda") for _ in range(2))
    late, nan, plain = 0, units - 1, units // 2
    amp = 16.0 / np.sqrt(d)                                       # a logit is amp times what a key's element 0 holds, and a random part
    q[late] *= 0.1
    k[late] *= 0.1
    q[late, :, 0], k[late, :, 0] = 16.0, -30.0 / amp
    k[late, 100:150, 0] = 30.0 / amp
    k[late, n - 40:, 0] = 60.0 / amp
    q, k = q.to(tdt), k.to(tdt)
    k[nan, 37, 5], k[nan, n - 1, 5], q[nan, 150, 3] = (float("nan"),) * 3
    out = torch.full((units + 1, n), -5.0, device="cuda")
    ssd.ssd_prefill_scores(q, k, units, n, d, dtype, out)
    assert bool((out[units] == -5.0).all()) and bool(torch.isfinite(out).all())
    ref = _scores_in_64_bits(q[[late, plain]], k[[late, plain]])
    z = q[nan].double() @ k[nan].double().T / np.sqrt(d)
    z = z.masked_fill(torch.isnan(z) | torch.ones((n, n), dtype=torch.bool, device="cuda").triu(1), -np.inf)
    for u, want, tol in ((late, ref[0], 64 * 2.0 ** -24 * 90.0), (plain, ref[1], 1e-5), (nan, torch.nan_to_num(torch.softmax(z, dim=-1)).sum(dim=0), 1e-5)):
        assert float(((out[u].double() - want).abs() / want.clamp_min(1e-3)).max()) < tol, u
    assert float(out[nan, 37]) == 0.0 and float(out[nan, n - 1]) == 0.0


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [40, 64, 128])
def test_prefill_scores_short_prompts_pass_a_logit_that_is_no_number_on(dtype, n):
    """Up to 128 tokens a query with such a logit makes the score of every key it attends to NaN; another unit keeps its own."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(n)
    q, k = (torch.randn((2, n, 64), generator=g).to(tdt) for _ in range(2))
    q[0, 20, 3] = float("nan")
    out = torch.empty((2, n), device="cuda")
    ssd.ssd_prefill_scores(q.cuda(), k.cuda(), 2, n, 64, dtype, out)
    got = out.cpu()
    assert bool(torch.isnan(got[0, :21]).all())
    _check_scores(got[1].numpy(), oracle.prefill_scores(q[1].float().numpy(), k[1].float().numpy(), 0.125), "the other unit")


def test_prefill_scores_bit_reproducible():
    g = torch.Generator().manual_seed(5)
    q = torch.randn((40, 200, 128), generator=g).to(torch.bfloat16).cuda()
    k = torch.randn((40, 200, 128), generator=g).to(torch.bfloat16).cuda()
    a = torch.empty((40, 200), device="cuda")
    b = torch.empty((40, 200), device="cuda")
    ssd.ssd_prefill_scores(q, k, 40, 200, 128, "bf16", a)
    ssd.ssd_prefill_scores(q, k, 40, 200, 128, "bf16", b)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_prefill_scores_equal_token_by_token_decode_accumulation():
    """Feeding the prompt one token at a time through the decode path with an unbounded budget accumulates the
    same scores (same definition, different kernels and summation order)."""
    n = 48
    wl = workload.Workload("pf-eq", L=1, prompts=1, H=4, d=128, dtype="bf16", n0=n, grid_h=1, grid_w=1, W=8, M=n + 2,
                           S=1, R=0, C=2, cadence=1, seed=77)
    ht = np.ones((1, 4), np.uint8)
    dev = {x: v.cuda() for x, v in workload.generate(wl, head_type=ht).items()}
    cache = make_cache(wl, ht)
    out = torch.empty((1, wl.B, wl.H, wl.d), dtype=torch.bfloat16, device="cuda")
    for p in range(n):
        ssd.ssd_decode_step(cache, 0, 1, dev["q"][p], dev["k"][p], dev["v"][p], out, True, True)
    pos, _, sc = [x.cpu().numpy() for x in cache.export(0)]
    Q = workload.dense_layout(dev["q"][:n]).contiguous()
    K = workload.dense_layout(dev["k"][:n]).contiguous()
    score = torch.empty((wl.B * wl.H, n), device="cuda")
    ssd.ssd_prefill_scores(Q, K, wl.B * wl.H, n, wl.d, "bf16", score)
    torch.cuda.synchronize()
    score = score.cpu().numpy().reshape(wl.B, wl.H, n)
    for b in range(wl.B):
        for h in range(wl.H):
            by_pos = {int(pp): float(ss) for pp, ss in zip(pos[b, h], sc[b, h]) if pp >= 0}
            assert sorted(by_pos) == list(range(n))
            _check_scores(np.array([by_pos[j] for j in range(n)], np.float32), score[b, h], "unit (%d,%d)" % (b, h))


@pytest.mark.parametrize("dtype,d,n0", [("bf16", 128, 64), ("f32", 64, 37)])
def test_prompt_pipeline_prefill_compress_decode(dtype, d, n0):
    """Prompt in one piece: scores from the prefill kernel, dense-source compression, then token-by-token
    decode of the image -- against an oracle that took the same route on its own scores."""
    wl = workload.Workload("pf-pipe", L=2, prompts=1, H=4, d=d, dtype=dtype, n0=n0, grid_h=3, grid_w=4, W=16, M=12,
                           S=1, R=1, C=3, cadence=2, seed=5 + n0)
    ht = workload.head_map(wl)
    data = workload.generate(wl, head_type=ht)
    dev = {x: v.cuda() for x, v in data.items()}
    Q = workload.dense_layout(dev["q"][:n0]).contiguous()
    K = workload.dense_layout(dev["k"][:n0]).contiguous()
    V = workload.dense_layout(dev["v"][:n0]).contiguous()
    n_units = wl.L * wl.B * wl.H
    score = torch.empty((wl.L, wl.B, wl.H, n0), device="cuda")
    ssd.ssd_prefill_scores(Q, K, n_units, n0, d, dtype, score)
    cache = make_cache(wl, ht)
    ssd.ssd_compress_kv(cache, 0, wl.L, K, V, score, n0)
    cache_first = {l: [x.cpu().numpy() for x in cache.export(l)] for l in range(wl.L)}     # right after the prompt's compression
    units = sample_units(wl, ht, 10 ** 9)
    sched = workload.compress_schedule(wl)
    steps = list(range(n0, wl.n_total))
    outs, exports, _ = gpu_decode(wl, dev, ht, sched, units, export_steps=steps, cache=cache, p_begin=n0)
    score_h = score.cpu().numpy()
    first_pos = {l: cache_first[l][0] for l in range(wl.L)}
    n_ties = 0
    for ui, (l, b, h) in enumerate(units):
        unit = (l, b, h)
        q_, K_, V_ = workload.unit_arrays(data, l, b, h)
        sem = ht[l, h] == workload.SEMANTIC
        ref_score = oracle.prefill_scores(q_[:n0], K_[:n0], wl.scale)
        _check_scores(score_h[l, b, h], ref_score, "prompt scores of %s" % (unit,))
        u = oracle.Unit(sem, wl.W, wl.S, wl.M, wl.R, wl.C)
        _, gap0 = u.load_dense(n0, ref_score)
        if sem:
            # the dense-source cut on the GPU's own prompt scores is the oracle's selection routine on those scores, always
            n_cand = n0 - min(wl.R, n0)
            keep, _ = oracle.top_m(score_h[l, b, h][:n_cand], np.arange(n_cand, dtype=np.int32), wl.M)
            got0 = sorted(int(x) for x in first_pos[l][b, h][: wl.M] if x >= 0)
            assert got0 == sorted(int(x) for x in keep), ("dense-source selection on the GPU's own scores", unit)
            hp, _, _, _ = u.state()
            if got0 != sorted(int(x) for x in hp):
                # the prompt cut itself fell the other way: excused only inside the rounding margin (its own-score
                # check is the assertion above); nothing further to compare
                assert 0 <= gap0 <= GAP_MARGIN, ("prompt cut differs above the tie margin", unit, gap0)
                n_ties += 1
                continue
        o_ref, hl, gl = u.run(q_, K_, V_, wl.scale, sched, log=True)
        div = compare_unit_sets(wl, ht, unit, l, exports, hl, gl, sched, p_begin=n0)
        upto = len(steps) if div is None else div[0] - n0 + 1
        check_outputs(outs[:upto, ui], o_ref[:upto], dtype, "unit %s after the prompt pipeline" % (unit,))
        if div is not None:
            n_ties += 1
            settle_near_tie(wl, dev, ht, sched, unit, l, exports, div[0], False)     # every step is exported with its "before" tables
    assert n_ties <= near_tie_cap(len(units))


# ---- classifier-free guidance mix (Eq. 1) -----------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,V", [(2, 1), (4, 7), (6, 64), (8, 1000), (128, 16384), (2, 16385)])
def test_cfg_mix_matches_oracle(dtype, B, V):
    say("cfg mix", dtype, B, V)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(B * 31 + V)
    p = (3.0 * torch.randn((B, V), generator=g)).to(tdt)
    out = torch.full((B // 2, V), -9.0, device="cuda")
    for gamma in (5.0, 0.0, -1.0):
        ssd.ssd_cfg_mix(p.cuda(), B, V, dtype, gamma, out)
        torch.cuda.synchronize()
        ref = oracle.cfg_mix(p.float().numpy(), gamma)
        got = out.cpu().numpy()
        # one fused multiply-add in fp32 on exactly representable inputs
        bound = 1e-6 * (np.abs(ref) + abs(gamma) * 6.0 + 1.0)
        assert (np.abs(got - ref) <= bound).all(), (gamma, float(np.abs(got - ref).max()))
        if gamma == 0.0:
            assert np.array_equal(got, p[0::2].float().numpy())


def _rows_are_the_sources(cache, K, V, pos):
    """Every row the one-layer cache holds, both planes of every unit, is the source's row of that slot's position, bit for
    bit.  pos: the exported table [B, H, slots]."""
    c = cache.cfg
    B, H, d, S = c.n_seqs, c.n_heads, c.head_dim, c.n_init_sink
    W, M = cache.layer_budget(0)
    sem = torch.from_numpy(cache.head_type[0] == ssd.SSD_SEMANTIC)
    base = (-cache.mem.data_ptr()) % 256
    off = base
    for kind, rows in ((False, S + W), (True, M + c.stage_cap)):
        heads = torch.nonzero(sem == kind).flatten().cuda()
        size = B * len(heads) * 2 * rows * d * K.element_size()
        units = cache.mem[off:off + size].view(K.dtype).view(B, len(heads), 2, rows, d)
        off = base + (off - base + size + 255) // 256 * 256
        at = pos[:, heads, :rows].long()
        for plane, src in ((0, K), (1, V)):
            want = torch.gather(src[:, heads], 2, at.clamp_min(0)[..., None].expand(-1, -1, -1, d))
            same = (units[:, :, plane] == want).all(dim=-1) | (at < 0)
            assert bool(same.all()), ("semantic" if kind else "spatial", "KV"[plane], torch.nonzero(~same)[:4].tolist())


def _dense_source_selection(B, H, n, scores, dtype="bf16", d=64, M=48, W=20, R=1, heads=False):
    from paper_2510_18716_amd.binding import make_config
    say("dense-source selection", B, H, n, scores, dtype, d, "M", M, "per-head", heads)
    S = 1
    g = torch.Generator(device="cuda").manual_seed(n)
    u = torch.rand((B, H, n), generator=g, device="cuda")
    score = {"spread": -torch.log(u.clamp_min(1e-6)), "few": (u * 5).floor() * 0.25, "equal": torch.full_like(u, 0.7),
             "zero": torch.zeros_like(u), "wide": torch.exp2(60 * u - 40)}[scores].contiguous()
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.randn((B, H, n, d), generator=g, device="cuda", dtype=tdt)
    V = torch.randn((B, H, n, d), generator=g, device="cuda", dtype=tdt)
    ht = np.zeros((1, H), np.uint8)
    ht[0, H // 2:] = ssd.SSD_SEMANTIC
    own = np.where(ht[0] == ssd.SSD_SEMANTIC, M, W)
    if heads:
        own = np.maximum(1, own - np.arange(H) % 5 * (own // 6))     # the first head of each type has the largest
        own[0], own[H // 2] = W, M
    cache = ssd.Cache(make_config(1, B, H, d, dtype, W, S, M, R, R + 2), ht, head_budget=own[None] if heads else None)
    ssd.ssd_compress_kv(cache, 0, 1, K, V, score, n)
    table = cache.export(0)
    _rows_are_the_sources(cache, K, V, table[0])
    pos, count, kept_score = (t.cpu().numpy() for t in table)
    sc = score.cpu().numpy()
    n_cand = n - min(n, R)
    for b in range(0, B, 7):
        for h in range(H):
            if h < H // 2:
                want = sorted(set(range(min(S, n))) | set(range(max(S, n - own[h]), n)))
                assert sorted(p for p in pos[b, h] if p >= 0) == want
            else:
                order = np.lexsort((np.arange(n_cand), -sc[b, h, :n_cand]))[:own[h]]
                heavy = sorted(int(i) for i in order)
                want = heavy + list(range(n_cand, n))
                assert [int(p) for p in pos[b, h][:len(heavy)]] == heavy
                assert [int(p) for p in pos[b, h][M:M + n - n_cand]] == want[len(heavy):]
                assert np.array_equal(kept_score[b, h][:len(heavy)], sc[b, h][heavy])
            assert count[b, h] == len(want)
    return cache, V, pos


@pytest.mark.parametrize("B,H", [(2, 4), (40, 16)])              # few units: a wide workgroup each; many: the narrow one
@pytest.mark.parametrize("n", [5, 64, 70, 257, 300, 1024, 1500, 4096])
@pytest.mark.parametrize("scores", ["spread", "few", "equal", "zero", "wide"])
def test_dense_source_selection_is_the_sorted_one(B, H, n, scores):
    """The kept set of the dense-source mode is what a sort by (score, lower position first) keeps, exactly, whatever the
    scores look like to a radix descent: long-tailed, a handful of distinct values, all equal, all zero, 60 binary
    orders of magnitude; the kept rows are the source's, bit for bit, in ascending order of position."""
    cache, V, pos = _dense_source_selection(B, H, n, scores)
    d = V.shape[-1]
    q = torch.zeros((1, B, H, d), dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    ssd.ssd_decode_attn(cache, 0, 1, q, out, False)               # zero query: the mean of the kept rows
    got = out.float().cpu().numpy()[0]
    for b in range(0, B, 7):
        Vb = V[b].float().cpu().numpy()
        for h in range(H):
            want = sorted(int(p) for p in pos[b, h] if p >= 0)
            np.testing.assert_allclose(got[b, h], Vb[h][want].mean(axis=0), atol=2e-2, rtol=1e-2)


@pytest.mark.parametrize("dtype,d,heads", [("bf16", 128, False), ("f32", 128, False), ("f32", 64, True), ("bf16", 128, True)])
@pytest.mark.parametrize("B,H", [(2, 4), (32, 16), (27, 19)])    # 512 units are the last few
@pytest.mark.parametrize("n,M,R", [(40, 48, 1), (256, 30, 0), (257, 48, 1), (257, 300, 1), (258, 48, 1), (260, 255, 8), (2049, 48, 1), (2050, 48, 1)])
def test_dense_source_at_the_edges_of_its_shapes(dtype, d, heads, B, H, n, M, R):
    """256 candidates (n - R), ranked by counting, and one more; a prompt just longer than that and kept whole; 2048 and one
    more; rows of 16 and of 32 fragments; budgets per head."""
    _dense_source_selection(B, H, n, "spread", dtype, d, M, W=20, R=R, heads=heads)


@pytest.mark.parametrize("B,H,n,dtype,d", [(80, 32, 40, "bf16", 128), (83, 31, 70, "bf16", 128), (83, 31, 33, "f32", 128), (128, 21, 65, "f32", 64),
                                             (80, 32, 64, "bf16", 128), (100, 32, 56, "bf16", 128), (100, 32, 57, "bf16", 128), (80, 32, 64, "f32", 128)])
def test_short_prompts_of_many_units(B, H, n, dtype, d):
    """From 2560 units of up to 32 KB on neighbouring units are dealt to one XCD (2560 and 2573: whole blocks of 512 and 13 beside them),
    and from 40 MB of keys on K is read without the hint unless rows of 256 bytes fill their tiles (57 of 64): the same scores (tolerance as for long prompts), the sorted selection."""
    _dense_source_selection(B, H, n, "spread", dtype, d, M=24, W=20)
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k = (torch.randn((B * H, n, d), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
    out = torch.full((B * H + 1, n), -5.0, device="cuda")
    ssd.ssd_prefill_scores(q, k, B * H, n, d, dtype, out)
    at = [0, 511, 512, B * H // 2, B * H - 1]
    ref = _scores_in_64_bits(q[at], k[at])
    assert bool((out[-1] == -5.0).all()) and bool(torch.isfinite(out).all())
    assert float(((out[at].double() - ref).abs() / ref.clamp_min(1e-3)).max()) < 1e-5


def _mix_case(n, V, dtype, gamma):
    """Against 64 bits; a row beyond the last must stay as it was.  Two roundings of fp32: of c - u, then of the result."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    p = torch.randn((2 * n, V), generator=torch.Generator(device="cuda").manual_seed(n + V), device="cuda").to(tdt)
    out = torch.full((n + 1, V), 7.0, device="cuda")
    ssd.ssd_cfg_mix(p, 2 * n, V, dtype, gamma, out)
    c, u = p.double()[0::2], p.double()[1::2]
    ref = c + gamma * (c - u)
    bound = 1.01 * 2.0 ** -24 * (abs(gamma) * (c - u).abs() + ref.abs())
    assert bool(((out[:n].double() - ref).abs() <= bound).all())
    assert bool((out[n] == 7.0).all())


@pytest.mark.parametrize("V", [3, 521])
def test_cfg_mix_more_prompts_than_one_grid_dimension_holds(V):
    """65536 is the first prompt a workgroup that has a row to itself (521: 66 pieces) reaches with its second stride; neither
    length keeps 16-byte alignment."""
    _mix_case(65537, V, "bf16", 2.5)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,V", [(1, 1), (3, 7), (85714, 7), (85715, 7), (150001, 4), (4099, 257), (9001, 67), (2333, 515), (601, 1030), (5, 8), (999, 8),
                                 (1001, 24), (70, 512), (67, 520), (33, 264), (7812, 512), (7813, 512), (7813, 513), (37, 1024), (37, 1032), (37, 516), (1, 600001),
                                 (2, 4 * 65537 * 4)])
def test_cfg_mix_short_rows_and_little_work(dtype, n, V):
    """Unaligned rows on both sides of 600000 elements in all (one element per lane; pieces), rows of 1 to 128 pieces that share
    a workgroup and of 129 that do not, bf16 rows of 64 on both sides of 4000000 elements in all, every remainder of a piece,
    a last workgroup with rows missing, rows longer than a grid's first pass."""
    say("cfg mix", dtype, n, V)
    _mix_case(n, V, dtype, 5.0)


@pytest.mark.parametrize("missing", [None, "_raw_stream", "_raw_device"])
def test_binding_takes_torchs_current_stream(missing, monkeypatch):
    """Also where torch does not have the accessors of the raw handle."""
    from paper_2510_18716_amd import binding
    from paper_2510_18716_amd.binding import _stream
    if missing:
        monkeypatch.setattr(binding, missing, None)
    side = torch.cuda.Stream()
    assert (_stream() or 0) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert _stream() == side.cuda_stream
    assert _stream(side) == side.cuda_stream and _stream(123) == 123
