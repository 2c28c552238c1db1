"""Logits rows that are not whole 16-byte pieces: odd vocabularies, row strides that leave the rows
2- or 4-byte aligned, bases that start inside a piece.  Chain (one work-group per sequence and
shared), per-sequence and tree samplers against the CPU oracle: tokens and counts exact on
sequences that the oracle does not flag.  Whatever lies between the rows and around the matrix holds
NaN (bf16 and fp32), so an element read past a row's end would show.
"""
import numpy as np
import pytest
import torch

import helpers
from helpers import compare_sampler, compare_tree_sampler, gpu_sample, gpu_tree_sample, oracle_sample, oracle_tree_sample
from paper_2510_26475_amd import binding, synth

pytestmark = pytest.mark.gpu

KS = [3, 0, 2, 1, 3, 2, 3, 0] * 4


def _wl(V, dtype, T):
    return synth.Workload("rows", B=0, k=0, Hq=1, Hkv=1, D=64, V=V, dtype=dtype, len_dist="uniform", len_lo=1, len_hi=1,
                          sigma=1.5, temperature=T)


def _spread(t, gap, shift):
    """The same rows `gap` elements further apart, starting `shift` elements into NaN."""
    rows, V = t.shape
    flat = torch.full((shift + rows * (V + gap) + 64,), float("nan"), dtype=t.dtype, device=t.device)
    view = flat[shift:shift + rows * (V + gap)].view(rows, V + gap)[:, :V]
    view.copy_(t)
    return view


# the last slot holds one element, one short of all, or is whole but unaligned; a vocabulary smaller
# than a slot; one slot and a bit; a part of a shared row that would hold the partial slot alone
SHAPES = [(8 * 300 + 1, 0, 0), (8 * 300 + 7, 0, 0), (2400, 1, 0), (2400, 0, 3), (1001, 3, 1), (9, 2, 0), (7, 1, 0), (3, 0, 0),
          (8 * 64 + 5, 0, 0), (50257, 0, 0)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [1.0, 1.3])
@pytest.mark.parametrize("V,gap,shift", SHAPES)
@pytest.mark.parametrize("split", [1, 2, 8])
def test_chain(oracle, V, gap, shift, dtype, T, split):
    wl = _wl(V, dtype, T)
    batch = synth.make_batch(wl, device="cuda", kv_lens=[k + 1 for k in KS], k_per_seq=KS, seed=V + split, with_attention=False)
    ref = oracle_sample(oracle, batch)
    batch.target_logits, batch.draft_logits = _spread(batch.target_logits, gap, shift), _spread(batch.draft_logits, gap, shift)
    with helpers.sampler_split(split):
        tally = compare_sampler(gpu_sample(batch), ref)
    assert tally["flagged"] <= max(3, 0.25 * len(KS)), tally


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,gap,shift", SHAPES)
def test_per_sequence_temperatures(oracle, V, gap, shift, dtype):
    wl = _wl(V, dtype, 1.0)
    batch = synth.make_batch(wl, device="cuda", kv_lens=[k + 1 for k in KS], k_per_seq=KS, seed=V, with_attention=False)
    temps = np.array([(0.0, 0.6, 1.0, 1.3)[b % 4] for b in range(len(KS))], dtype=np.float32)
    for b, qi in enumerate(batch.q_indptr.tolist()[:-1]):  # a tie that straddles the last slot, greedy rows
        if temps[b] == 0:
            batch.target_logits[qi, V - 1] = batch.target_logits[qi, V // 2] = 40.0
    odt = oracle.F32 if dtype == "f32" else oracle.BF16
    ref = oracle.rejection_sample_per_seq(
        synth.to_host_array(batch.target_logits), synth.to_host_array(batch.draft_logits), batch.draft_tokens.cpu().numpy(),
        batch.q_indptr.cpu().numpy(), batch.u_accept.cpu().numpy(), batch.u_final.cpu().numpy(), batch.max_k, temps, odt)
    target, draft = _spread(batch.target_logits, gap, shift), _spread(batch.draft_logits, gap, shift)
    B = len(KS)
    toks = torch.full((B, batch.max_k + 1), -7, dtype=torch.int32, device="cuda")
    n, flags = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    binding.respec_rejection_sample_per_seq(target, draft, batch.draft_tokens, batch.q_indptr, batch.u_accept, batch.u_final,
                                            torch.from_numpy(temps).cuda(), toks, n, flags, batch.max_k)
    torch.cuda.synchronize()
    compare_sampler((toks.cpu().numpy(), n.cpu().numpy(), flags.cpu().numpy()), ref)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [1.0, 1.3])
@pytest.mark.parametrize("V,gap,shift", SHAPES)
def test_tree(oracle, V, gap, shift, dtype, T):
    parents = [synth.caterpillar_parents(2, 3), [-1, 0, 0], [-1], [-1, 0, 1, 2]] * 6
    tb = synth.make_tree_batch(_wl(V, dtype, T), parents, device="cuda", kv_lens=[len(p) for p in parents], seed=V, with_attention=False)
    ref = oracle_tree_sample(oracle, tb)
    tb.target_logits, tb.draft_logits = _spread(tb.target_logits, gap, shift), _spread(tb.draft_logits, gap, shift)
    compare_tree_sampler(gpu_tree_sample(tb), ref)


# The guarded form (running references per thread) on the same rows: it too must not count on rows
# that start on 16 bytes
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,gap,shift", SHAPES)
@pytest.mark.parametrize("split", [1, 2])
def test_guarded_form(oracle, V, gap, shift, dtype, split):
    wl = _wl(V, dtype, 1.3)
    batch = synth.make_batch(wl, device="cuda", kv_lens=[k + 1 for k in KS], k_per_seq=KS, seed=V + split, with_attention=False)
    parents = [synth.caterpillar_parents(2, 3), [-1, 0, 0], [-1], [-1, 0, 1, 2]] * 6
    tb = synth.make_tree_batch(wl, parents, device="cuda", kv_lens=[len(p) for p in parents], seed=V, with_attention=False)
    ref, tree_ref = oracle_sample(oracle, batch), oracle_tree_sample(oracle, tb)
    for t in (batch, tb):
        t.target_logits, t.draft_logits = _spread(t.target_logits, gap, shift), _spread(t.draft_logits, gap, shift)
    with helpers.sampler_split(split), helpers.env_setting("RESPEC_SAMPLER_GUARDED", 1):
        compare_sampler(gpu_sample(batch), ref)
        compare_tree_sampler(gpu_tree_sample(tb), tree_ref)


# Short rows are taken eight positions at a time: what lies behind a rejected position is read and must
# not matter (10 drafts: two groups of positions)
@pytest.mark.parametrize("dtype,V", [("bf16", 1000), ("f32", 1001), ("f32", 2048), ("f32", 4096)])
@pytest.mark.parametrize("T", [1.0, 1.3])
def test_rows_behind_a_rejection_of_a_short_row_may_hold_anything(oracle, dtype, V, T):
    ks = [10, 9, 8, 7, 1, 0] * 5
    batch = synth.make_batch(_wl(V, dtype, T), device="cuda", kv_lens=[k + 1 for k in ks], k_per_seq=ks, seed=V, with_attention=False)
    batch.draft_logits.copy_((batch.target_logits[[q for b, k in enumerate(ks) for q in range(int(batch.q_indptr[b]), int(batch.q_indptr[b]) + k)]]
                              .float() + 0.1 * torch.randn_like(batch.draft_logits.float())).to(batch.draft_logits.dtype))
    ref = oracle_sample(oracle, batch)
    clean = gpu_sample(batch, workspace=None)
    compare_sampler(clean, ref)
    assert clean[1].max() >= 8                     # a chain that reaches the second group
    qi = batch.q_indptr.tolist()
    for b, k in enumerate(ks):
        n = int(clean[1][b])
        if n < k:
            batch.target_logits[qi[b] + n + 1:qi[b + 1]] = float("nan")
            batch.draft_logits[qi[b] - b + n + 1:qi[b + 1] - (b + 1)] = float("nan")
    poisoned = gpu_sample(batch, workspace=None)
    for x, y in zip(clean, poisoned):
        np.testing.assert_array_equal(x, y)


def _two_heavy_tokens(first, last, V, B, T, k, seed):
    """B row blocks (k + 1 rows of V fp32 logits) whose last row holds its mass in two tokens about
    84 T above the rest, between the indices first and last: nearly the largest distance at which a
    weight against the rest's level is finite in binary32.  Returns (target rows, the indices, the share
    of the first heavy token)."""
    gen = torch.Generator().manual_seed(seed)
    rows = torch.randn((B * (k + 1), V), generator=gen)
    level = rows[k::k + 1].amax(1)
    at = torch.sort(first + torch.rand((B, 2), generator=gen).mul(last - first - 1).long(), dim=1).values
    at[:, 1] = torch.maximum(at[:, 1], at[:, 0] + 1)
    z = (level[:, None] + T * (84.0 + torch.rand((B, 2), generator=gen))).float()
    rows[torch.arange(k, B * (k + 1), k + 1)[:, None], at] = z
    share = 1.0 / (1.0 + torch.exp((z[:, 1].double() - z[:, 0].double()) / float(np.float32(T))))
    return rows, at, share.numpy()


def _compare_forms(form, batch, ref):
    """The batch through one form of the samplers (a tree of root nodes for "tree") against the oracle."""
    B, k, T, V = len(batch.k_per_seq), batch.max_k, batch.wl.temperature, batch.wl.V
    if form == "tree":
        tb = synth.make_tree_batch(batch.wl, [list(range(-1, k))] * B, device="cuda", kv_lens=[k + 1] * B, seed=1, with_attention=False)
        tb.target_logits.copy_(batch.target_logits)
        tb.u_final.copy_(batch.u_final)
        if k:  # (k = 1: the root's row pair, the leaf's target row)
            tb.draft_logits[0::2] = batch.draft_logits
            tb.node_tokens[1::2] = batch.draft_tokens
            tb.u_accept[1::2] = batch.u_accept
        toks, _, n, flags = gpu_tree_sample(tb)
        compare_sampler((toks, n, flags), ref)
    elif form == "per sequence":
        toks = torch.full((B, k + 1), -7, dtype=torch.int32, device="cuda")
        n, flags = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        binding.respec_rejection_sample_per_seq(batch.target_logits, batch.draft_logits, batch.draft_tokens, batch.q_indptr,
                                                batch.u_accept, batch.u_final, torch.full((B,), T, device="cuda"), toks, n, flags, k)
        torch.cuda.synchronize()
        compare_sampler((toks.cpu().numpy(), n.cpu().numpy(), flags.cpu().numpy()), ref)
    else:
        with helpers.sampler_split(1 if form == "one work-group" else 2), helpers.env_setting("RESPEC_SAMPLER_TWO_ITEMS", int(form == "two items")):
            toks, n, flags = gpu_sample(batch)
        compare_sampler((toks, n, flags), ref)
        return toks, n, flags
    return (toks, n, flags) if isinstance(toks, np.ndarray) else (toks.cpu().numpy(), n.cpu().numpy(), flags.cpu().numpy())


# A weight 121 binary orders above the reference that it is formed against has an exponent rounded to
# 2^-18, so the edge between two such tokens can be off by 1.3e-6, more than the band that is flagged.
# Uniforms just outside the band show it (in 1 to 2 % of the rows).  The heavy tokens lie behind the
# first 512 slots and within the first 2048 (1024 in a part of a shared row).
@pytest.mark.parametrize("T", [0.85, 1.3])
@pytest.mark.parametrize("form", ["one work-group", "shared", "per sequence", "tree"])
def test_draws_with_64_bit_weights_look_as_far_for_their_reference_as_a_normaliser_pass(oracle, form, T):
    V, B, k = (8192, 128, 1) if form == "shared" else (8192, 1024, 0)
    rows, _, share = _two_heavy_tokens(4 * 512, 4 * (1024 if k else 2048), V, B, T, k, seed=int(100 * T))
    batch = synth.make_batch(_wl(V, "f32", T), device="cuda", kv_lens=[k + 1] * B, k_per_seq=[k] * B, seed=1, with_attention=False)
    batch.target_logits.copy_(rows)
    if k:
        batch.draft_logits.copy_(rows[0::2])
        batch.u_accept.mul_(0.999)
    batch.u_final.copy_(torch.from_numpy((share + np.where(np.arange(B) % 2, 1.05e-6, -1.05e-6)).astype(np.float32)))
    ref = oracle_sample(oracle, batch)
    assert (ref[2] != 0).sum() <= B // 8
    _compare_forms(form, batch, ref)


# The same distance in rows that are not whole aligned slots, heavy tokens anywhere: these rows had the
# guarded pass, which moves its reference, and must not do worse in the fast ones.  Draws at the edge
# between the two tokens, and acceptance tests of the first of them (its share is exact here, the sum
# it is divided by is what can be off).
@pytest.mark.parametrize("T", [0.6, 1.3])
@pytest.mark.parametrize("what", ["draw", "accept"])
@pytest.mark.parametrize("form", ["one work-group", "shared", "per sequence", "tree"])
def test_heavy_tokens_far_behind_the_start_of_an_odd_row(oracle, form, what, T):
    V, B, k = 50257, 128, 1
    rows, at, share = _two_heavy_tokens(4 * 2100, 4 * 6200, V, B, T, k, seed=int(100 * T))
    side = np.where(np.arange(B) % 2, 1.05e-6, -1.05e-6)
    wl = _wl(V, "f32", T)
    batch = synth.make_batch(wl, device="cuda", kv_lens=[k + 1] * B, k_per_seq=[k] * B, seed=1, with_attention=False)
    batch.target_logits.copy_(rows)
    if what == "draw":
        batch.draft_logits.copy_(rows[0::2])  # every draft is accepted, the heavy row is the bonus row
        batch.u_accept.mul_(0.999)
        batch.u_final.copy_(torch.from_numpy((share + side).astype(np.float32)))
    else:
        batch.target_logits.copy_(rows.view(B, 2, V).flip(1).reshape(2 * B, V))  # the heavy row is the draft's
        q = torch.randn((B, V), generator=torch.Generator().manual_seed(3))
        ar, x, T64 = torch.arange(B), at[:, 0], float(np.float32(T))
        rest = torch.exp(q.double() / T64).sum(1) - torch.exp(q[ar, x].double() / T64)
        q[ar, x] = (T64 * torch.log(3.0 * rest)).float()  # q(x) about 0.75
        qx = 1.0 / (1.0 + rest * torch.exp(-q[ar, x].double() / T64)).numpy()
        batch.draft_logits.copy_(q)
        batch.draft_tokens.copy_(x.to(torch.int32))
        batch.u_accept.copy_(torch.from_numpy((share / qx + side).astype(np.float32)))
    ref = oracle_sample(oracle, batch)
    assert (ref[2] != 0).sum() <= B // 8
    if what == "accept":
        assert B // 5 < ref[1].sum() < B  # (uniforms above 1 among them: never accepted)
    _compare_forms(form, batch, ref)


# Four tokens 27.5 T (39.7 binary orders) above the rest of a row, in the slots of four threads of one region: no thread's
# sum calls for the guarded pass, and the sum over the row is 2^41.7 of its reference.  A draw that has the
# normaliser (the residual's, and the second of a bonus row's two) has to take such a total for what it is.  (The
# slots lie behind the first batch of every form: 2048 slots of a row or of the second half of a shared one.)
@pytest.mark.parametrize("T,above", [(1.0, 27.5), (0.4, 11.0)])
@pytest.mark.parametrize("what", ["bonus", "residual"])
@pytest.mark.parametrize("form", ["one work-group", "shared", "two items", "per sequence", "tree"])
@pytest.mark.parametrize("dtype,V,gap,slot", [("f32", 50257, 0, 8836), ("bf16", 50257, 0, 5700), ("f32", 50256, 1, 8836)])
def test_tokens_just_inside_the_range_of_a_reference(oracle, dtype, V, gap, slot, form, what, T, above):
    B, epv = 32, 8 if dtype == "bf16" else 4
    gen = torch.Generator().manual_seed(V + slot)
    rows = -0.5 - torch.rand((2 * B, V), generator=gen)
    rows[:, ::64] = 0.0                           # every wave's reference
    heavy = [epv * (slot + j) + j % epv for j in range(4)]
    hot = slice(1, None, 2) if what == "bonus" else slice(0, None, 2)
    rows[hot, heavy] = above
    batch = synth.make_batch(_wl(V, dtype, T), device="cuda", kv_lens=[2] * B, k_per_seq=[1] * B, seed=1, with_attention=False)
    batch.target_logits.copy_(rows)
    batch.draft_logits.copy_(rows[0::2] if what == "bonus" else rows[1::2])
    batch.draft_tokens.fill_(7)
    batch.u_accept.fill_(0.5)                     # p = q: accepted; p(7) a millionth of q(7): rejected
    batch.u_final.copy_((torch.arange(B) + 0.5) / B)
    ref = oracle_sample(oracle, batch)
    assert not ref[2].any() and (ref[1] == (1 if what == "bonus" else 0)).all()
    if gap:
        batch.target_logits, batch.draft_logits = _spread(batch.target_logits, gap, 0), _spread(batch.draft_logits, gap, 0)
    got = _compare_forms(form, batch, ref)
    drawn = got[0][np.arange(B), got[1]]
    assert set(drawn.tolist()) == set(heavy)      # (nothing else has a millionth of the mass, flagged or not)


# Waves whose first slots hold no finite logit have no reference of their own, and most of the row's mass far below 1 in their
# later ones (120 T: an exponential against 0 is less than binary32 has).  Acceptance tests at half and at twice the ratio; the sum
# without those slots is a quarter of the row's.
@pytest.mark.parametrize("T", [1.0, 1.3])
@pytest.mark.parametrize("form", ["one work-group", "shared", "two items", "per sequence", "tree"])
@pytest.mark.parametrize("dtype,odd", [("f32", 0), ("bf16", 0), ("f32", 1)])
def test_waves_without_a_finite_logit_in_their_first_slots(oracle, dtype, odd, form, T):
    B, epv, T64 = 32, 8 if dtype == "bf16" else 4, float(np.float32(T))
    V = epv * 8192 + odd
    gen = torch.Generator().manual_seed(V)
    slot = torch.arange(V) // epv
    wave = slot % 256 < 64                        # of the first batches of every form: all of their slots, and others
    target = torch.randn((2 * B, V), generator=gen) - 120.0 * T64
    target[:, wave] += 3.0 * T64
    target[0::2, wave & (slot % 4096 < 2048)] = float("-inf")
    draft = torch.randn((B, V), generator=gen)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    target, draft = target.to(dt), draft.to(dt)
    zp, zq = target[0::2].double() / T64, draft.double() / T64
    ratio = torch.exp((zp - zp.logsumexp(1, keepdim=True)) - (zq - zq.logsumexp(1, keepdim=True)))
    x = ((ratio > 0.1) & (ratio < 0.45)).int().argmax(1)
    rho = ratio[torch.arange(B), x]
    batch = synth.make_batch(_wl(V, dtype, T), device="cuda", kv_lens=[2] * B, k_per_seq=[1] * B, seed=1, with_attention=False)
    batch.target_logits.copy_(target)
    batch.draft_logits.copy_(draft)
    batch.draft_tokens.copy_(x.to(torch.int32))
    batch.u_accept.copy_(torch.where(torch.arange(B) % 2 == 0, 0.5 * rho, 2.0 * rho))
    ref = oracle_sample(oracle, batch)
    assert (ref[1] == (np.arange(B) + 1) % 2).all() and (ref[2] != 0).sum() <= B // 8
    _compare_forms(form, batch, ref)


# Short rows are summed by one wave, long ones by the block; neither may be the less exact one.  The
# acceptance test is taken in 64 bits, so uniforms one binary32 step from the ratio show the error of
# the normalisers: their sums over 2048 elements are good to about 3e-9 (exp2's last bit, averaged over
# the heavy tokens), so at relative distances of 1.5e-8 and more (three deviations of two such sums)
# less than one in a hundred falls on the wrong side; the block's sums put up to 1.7 % there, binary32
# accumulators of up to eight terms per lane 3 to 9 %.
@pytest.mark.parametrize("dtype,V", [("f32", 2048), ("f32", 1999), ("bf16", 4096)])
@pytest.mark.parametrize("T", [1.0, 1.3])
def test_normalisers_of_short_rows_are_as_exact_as_those_of_long_ones(dtype, V, T):
    B, k, T64 = 2048, 2, float(np.float32(T))
    batch = synth.make_batch(_wl(V, dtype, T), device="cuda", kv_lens=[k + 1] * B, k_per_seq=[k] * B, seed=V, with_attention=False)
    zp, zq = batch.target_logits[0::3].double().cpu() / T64, batch.draft_logits[0::2].double().cpu() / T64
    ratio = torch.exp((zp - zp.logsumexp(1, keepdim=True)) - (zq - zq.logsumexp(1, keepdim=True)))
    x = ((ratio > 0.5) & (ratio < 1.0)).int().argmax(1)
    rho = ratio[torch.arange(B), x].numpy()
    u = rho.astype(np.float32)
    above = np.arange(B) % 2 == 1
    wrong_side = (u.astype(np.float64) > rho) != above
    u = np.where(wrong_side, np.nextafter(u, np.where(above, np.float32(2), np.float32(0)), dtype=np.float32), u)
    batch.draft_tokens[0::2] = x.to(torch.int32).cuda()
    batch.u_accept[0::2] = torch.from_numpy(u).cuda()
    n = gpu_sample(batch, workspace=None)[1]
    far = (np.abs(u.astype(np.float64) - rho) >= 1.5e-8 * rho) & (rho > 0.5) & (rho < 1.0)
    assert far.sum() > B // 2
    wrong = ((n > 0) == above) & far
    print(f"{wrong.sum()} of {far.sum()} on the wrong side")
    assert wrong.sum() <= 0.01 * far.sum()


# Shared sequences stream two chain items as one run of batches (256 threads, four slots each): an item of one batch, of
# exactly one, of two and three, a last batch of a slot; chains that end on either item, or on the bonus row.
# Item two of some sequences overflows its reference (an outlier far above its first batch), or has no finite logit there.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [1.0, 1.3])
@pytest.mark.parametrize("slots", [1984, 2048, 2112, 4096, 4160, 6144, 6200])
@pytest.mark.parametrize("short", [0, 1])
def test_two_items_of_a_shared_chain_are_one_stream(oracle, slots, short, dtype, T):
    V = slots * (8 if dtype == "bf16" else 4) - short
    batch = synth.make_batch(_wl(V, dtype, T), device="cuda", kv_lens=[k + 1 for k in KS], k_per_seq=KS, seed=slots + short, with_attention=False)
    for b, qi in enumerate(batch.q_indptr.tolist()[:-1]):
        if KS[b] == 3 and b % 8 == 0:
            batch.target_logits[qi + 1, V - 3] = 250.0
        if KS[b] == 2 and b % 8 == 2:
            batch.target_logits[qi + 2, :V // 2 + 64] = float("-inf")
    ref = oracle_sample(oracle, batch)
    with helpers.sampler_split(2):
        tally = compare_sampler(gpu_sample(batch), ref)
    assert tally["flagged"] <= max(3, 0.25 * len(KS)), tally


# The region totals of a shared draw are searched by one scan over a wave: crossings in every region, none below, and
# regions without mass in between
@pytest.mark.parametrize("split", [1, 2, 4, 8])
@pytest.mark.parametrize("T", [1.0, 1.3])
def test_crossings_in_every_region(oracle, split, T):
    ks, V = [0] * 32, 8 * 64 * 32
    batch = synth.make_batch(_wl(V, "bf16", T), device="cuda", kv_lens=[1] * 32, k_per_seq=ks, seed=split, with_attention=False)
    for b in range(32):
        if b % 2:  # mass in every third region of 64 slots only
            keep = (torch.arange(V, device="cuda") // 512) % 3 == b % 3
            batch.target_logits[b, ~keep] = float("-inf")
        batch.u_final[b] = (b + 0.5) / 32 if b < 30 else (0.0, 1.0 - 2.0 ** -24)[b - 30]
    ref = oracle_sample(oracle, batch)
    with helpers.sampler_split(split):
        tally = compare_sampler(gpu_sample(batch), ref)
    assert tally["flagged"] <= 6, tally   # (the uniforms 0 and 1 - 2^-24, and a quarter of a boundary draw per row or so)


# Masked vocabularies: the finite logits of a row lie in one stretch (its start, its end, across the middle, one token), of a
# target row and its drafter's row not always in the same, so that some parts of a shared row have none.  A part
# of one batch of its work-group, of two, of three; odd rows, whose last part may hold nothing but the partial slot.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [1.0, 1.3])
@pytest.mark.parametrize("slots,split", [(1024, 2), (4096, 4), (2048, 2), (4096, 2), (6200, 2)])
@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("two_items", [0, 1])
def test_parts_without_a_finite_logit(oracle, two_items, odd, slots, split, T, dtype):
    V = slots * (8 if dtype == "bf16" else 4) + odd
    batch = synth.make_batch(_wl(V, dtype, T), device="cuda", kv_lens=[k + 1 for k in KS], k_per_seq=KS, seed=slots, with_attention=False)
    keep = [slice(0, V // 6), slice(V - V // 7, V), slice(V // 2 - 100, V // 2 + 2000), slice(V - 1, V), slice(0, V), slice(3, 4)]
    draft_row = 0
    for b, qi in enumerate(batch.q_indptr.tolist()[:-1]):
        for i in range(KS[b] + 1):
            t, kept = batch.target_logits[qi + i], keep[(b + 5 * i) % 6]
            finite = t[kept].clone()
            t.fill_(float("-inf"))
            t[kept] = finite
            if i < KS[b]:
                q = batch.draft_logits[draft_row]
                if b % 3:                      # (b % 3 == 0: the drafter's row is not masked)
                    q[torch.isinf(t)] = float("-inf")
                if b % 2:                      # a token that the target allows
                    batch.draft_tokens[draft_row] = int(torch.argmax(t.float()))
                draft_row += 1
    ref = oracle_sample(oracle, batch)
    with helpers.sampler_split(split), helpers.env_setting("RESPEC_SAMPLER_TWO_ITEMS", two_items):
        tally = compare_sampler(gpu_sample(batch), ref)
    assert tally["flagged"] <= 0.25 * len(KS), tally


def _timer(batch):
    """A function that times the batch's call: the median of seven runs of forty calls, us."""
    B, k = len(batch.k_per_seq), batch.max_k
    dt = binding.RESPEC_F32 if batch.target_logits.dtype == torch.float32 else binding.RESPEC_BF16
    ws = helpers.sampler_workspace(B, batch.wl.V, dt, "cuda")
    out = torch.empty((B, k + 1), dtype=torch.int32, device="cuda")
    n, flags = (torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(2))

    def us_per_call():
        times = []
        for _ in range(7):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(40):
                binding.respec_rejection_sample(batch.target_logits, batch.draft_logits, batch.draft_tokens, batch.q_indptr, batch.u_accept,
                                                batch.u_final, out, n, flags, k, batch.wl.temperature, workspace=ws)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end) / 40 * 1e3)
        return sorted(times)[3]

    return us_per_call


# Rows that one work-group takes as fast are not shared (these were, and took 1.15 to 1.3 times as long).
@pytest.mark.parametrize("dtype,V,B", [("f32", 8192, 64), ("f32", 12288, 4), ("bf16", 12288, 4), ("bf16", 16384, 64)])
def test_short_rows_are_shared_only_where_that_is_no_slower(dtype, V, B):
    batch = synth.make_batch(_wl(V, dtype, 1.0), device="cuda", kv_lens=[4] * B, k_per_seq=[3] * B, seed=1, with_attention=False)
    us_per_call = _timer(batch)
    us_per_call()
    chosen = us_per_call()
    with helpers.sampler_split(1):
        alone = us_per_call()
    print(f"{chosen:.1f} us, by one work-group {alone:.1f}")
    assert chosen <= 1.1 * alone


# Such a part used to make every part of its sequence repeat its passes one by one: 83 us against 24 of an unmasked call, and 28
# of one work-group.  (24 us now; the bound leaves room for a busy device.)
def test_a_masked_vocabulary_does_not_slow_a_shared_sequence():
    B, V, k = 64, 32000, 4
    batch = synth.make_batch(_wl(V, "bf16", 1.0), device="cuda", kv_lens=[k + 1] * B, k_per_seq=[k] * B, seed=1, with_attention=False)
    us_per_call = _timer(batch)
    us_per_call()
    plain = us_per_call()
    batch.target_logits[:, V // 6:] = float("-inf")
    batch.draft_logits[:, V // 6:] = float("-inf")
    batch.draft_tokens.copy_(torch.multinomial(torch.softmax(batch.draft_logits.float(), 1), 1)[:, 0])
    masked = us_per_call()
    print(f"{plain:.1f} us, masked {masked:.1f} us")
    assert masked <= 2.0 * plain


# A stage's mark has ten bits.  With three exchanges per position (each of these has a part without finite logits, but the first
# two) a chain of 342 drafts left words in the mailbox with the mark of the next call's first stage.
def test_a_long_chain_leaves_no_words_that_the_next_call_could_take(oracle):
    V, k = 8 * 64 * 8, 342
    batch = synth.make_batch(_wl(V, "bf16", 1.0), device="cuda", kv_lens=[k + 1], k_per_seq=[k], seed=3, with_attention=False)
    batch.target_logits[2:, V // 2:] = float("-inf")
    batch.draft_logits.copy_(batch.target_logits[:k])
    batch.draft_tokens.copy_(torch.argmax(batch.target_logits[:k].float(), 1))
    ws = torch.zeros(binding.respec_rejection_sample_workspace_bytes(1, k + 1, V, binding.RESPEC_BF16), dtype=torch.uint8, device="cuda")
    for u, accepted in ((0.5, k), (1.5, 0), (0.5, k)):    # (identical rows: every draft is accepted; above 1: none)
        batch.u_accept.fill_(u)
        ref = oracle_sample(oracle, batch)
        assert ref[1][0] == accepted
        with helpers.sampler_split(2), helpers.env_setting("RESPEC_SAMPLER_TWO_ITEMS", 1):
            got = gpu_sample(batch, workspace=ws)
        assert got[1][0] == accepted
        compare_sampler(got, ref)
