"""Sequences shared without a workspace where a part cannot go by what the others see: parts without a finite logit, largest
logits that tie across parts, passes that overflow in one part, residuals that come out empty, and calls that end early or overlap.
Against the CPU oracle, met and alone; where the oracle flags a draw, against one work-group per sequence."""
import numpy as np
import pytest
import torch

from helpers import compare_sampler, compare_tree_sampler, env_setting, gpu_tree_sample, oracle_tree_sample
from paper_2510_26475_amd import binding, synth
from test_gpu_sampler_claim import _Call, _chain, _tree, _wl

pytestmark = pytest.mark.gpu

TREES = [[-1, 0, 0], [-1, 0, 1], [-1], [-1, 0, 0, 0], [-1, 0, 1, 1], [-1, 0, 1, 2, 3]]
MASKED = 77  # a token that neither row of an "empty" pair allows


def _edit(what, pairs, target, draft):
    """Makes the rows (t, d; d None: no drafter row) of a batch into what the case is about."""
    V = target.shape[1]
    for i, (t, d) in enumerate(pairs):
        p, q = target[t], draft[d] if d is not None else None
        if what == "masked":  # finite logits in one or two of the parts only
            keep = [slice(V // 2 + 9, V // 2 + V // 5), slice(V - V // 9, V), slice(0, V // 6), slice(V // 4 - 50, V // 4 + 50), slice(V - 1, V)][i % 5]
            for row in (p, q) if q is not None and i % 3 else (p,):
                finite = row[keep].clone()
                row.fill_(float("-inf"))
                row[keep] = finite
        elif what == "outliers":  # far above every reference taken from a row's or a part's start
            if i % 2:
                p[V - 3 - i % 1000] = 200.0 + i % 7
            if q is not None and i % 3 == 0:
                q[5 * V // 8 + i] = 150.0
            if i % 4 == 2:
                p[V // 2 + V // 3] = 60.0
        elif what == "empty":  # equal rows, and a draft token of no mass
            if q is not None:
                q.copy_(p)
                p[MASKED] = q[MASKED] = float("-inf")
        else:
            raise ValueError(what)


def _equal(got, want):
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


# whole and ragged rows, parts of four and of two (one and two items per stage)
SIZES = [(24, 151936, "bf16"), (24, 100003, "bf16"), (100, 65536, "bf16"), (24, 80001, "f32")]


@pytest.mark.parametrize("what", ["masked", "outliers", "empty"])
@pytest.mark.parametrize("B,V,dtype", SIZES)
def test_temperatures(oracle, B, V, dtype, what):
    batch, temps = _chain(B, 3, V, dtype, seed=B + 1)
    pairs, q0 = [], batch.q_indptr.tolist()
    for b, k in enumerate(batch.k_per_seq):
        pairs += [(q0[b] + i, q0[b] - b + i if i < k else None) for i in range(k + 1)]
    _edit(what, pairs, batch.target_logits, batch.draft_logits)
    for b, k in enumerate(batch.k_per_seq):
        for i in range(k):
            row = q0[b] - b + i
            if what == "empty":
                batch.draft_tokens[row] = MASKED if (b + i) % 2 else int(batch.draft_logits[row].float().argmax())
            elif b % 2:  # a token that the target allows
                batch.draft_tokens[row] = int(batch.target_logits[q0[b] + i].float().argmax())
    call = _Call(batch, temps)
    ref = call.reference(oracle)
    with env_setting("RESPEC_SAMPLER_CLAIM", 0):
        call()
        alone = [a.copy() for a in call.result()]
    compare_sampler(alone, ref)
    for ticks in (None, -1, 0):
        with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks):
            call()
        got = call.result()
        compare_sampler(got, ref)
        if what == "empty":
            _equal(got, alone)
    assert len(set(ref[1].tolist())) >= 2 and (what != "empty" or (alone[2] & 2).sum() >= B // 4)


@pytest.mark.parametrize("what", ["masked", "outliers", "empty"])
@pytest.mark.parametrize("B,V,dtype,T", [(24, 151936, "bf16", 0.6), (24, 100003, "bf16", 1.0), (100, 131072, "bf16", 1.3), (24, 80001, "f32", 0.6)])
def test_trees(oracle, B, V, dtype, T, what):
    tb = synth.make_tree_batch(_wl(B, 4, V, dtype, T), [TREES[b % 6] for b in range(B)], device="cuda", kv_lens=[64] * B, seed=B, with_attention=False)
    q0, pairs = tb.q_indptr.tolist(), []
    for b, par in enumerate(tb.parents_per_seq):
        inner = set(par)
        pairs += [(q0[b] + i, q0[b] + i if i in inner else None) for i in range(len(par))]
    _edit(what, pairs, tb.target_logits, tb.draft_logits)
    for b, par in enumerate(tb.parents_per_seq):
        for i in range(1, len(par)):
            row, of = q0[b] + i, q0[b] + par[i]
            if what == "empty":
                tb.node_tokens[row] = MASKED if (b + i) % 3 else int(tb.draft_logits[of].float().argmax())
            elif (b + i) % 2:
                tb.node_tokens[row] = int(tb.target_logits[of].float().argmax())
    ref = oracle_tree_sample(oracle, tb)
    with env_setting("RESPEC_SAMPLER_CLAIM", 0):
        alone = gpu_tree_sample(tb)
    compare_tree_sampler(alone, ref)
    for ticks in (None, -1, 0):
        with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks):
            got = gpu_tree_sample(tb)
        compare_tree_sampler(got, ref)
        if what == "empty" and dtype == "bf16" and T == 0.6:
            # (a tree's 64-bit weights are differences of rounded products: where they cancel, what is left of them is drawn from)
            _equal(got, alone)
    assert len(set(ref[2].tolist())) >= 2 and (what != "empty" or (ref[3] & 2).sum() >= B // 4)


# Greedy sequences take the lowest of equal largest logits, wherever the parts' borders lie: exactly, no draw is flagged.
@pytest.mark.parametrize("B,V,dtype", SIZES)
def test_greedy_ties_across_parts(oracle, B, V, dtype):
    k = [3, 1, 0, 3]
    batch = synth.make_batch(_wl(B, 3, V, dtype), device="cuda", kv_lens=[64] * B, k_per_seq=[k[b % 4] for b in range(B)], seed=2, with_attention=False)
    top = (batch.target_logits.float().max() + 1).to(batch.target_logits.dtype)
    q0, epv = batch.q_indptr.tolist(), 8 if dtype == "bf16" else 4
    slots = (V + epv - 1) // epv
    borders = [part * (((slots + n - 1) // n + 63) // 64 * 64) * epv for n in (2, 4) for part in range(1, n)]  # first elements of parts
    places = [x + e for x in sorted(set(borders)) for e in (-1, 0, 1)] + [0, V - 1]
    for b in range(B):
        for i in range(k[b % 4] + 1):
            row = batch.target_logits[q0[b] + i]
            chosen = [places[(3 * b + 5 * i + j * 7) % len(places)] for j in range(1 + (b + i) % 4)]
            row[chosen] = top
            if i < k[b % 4]:  # the first of them, or (not accepted) the last
                batch.draft_tokens[q0[b] - b + i] = min(chosen) if (b + i) % 5 else max(chosen)
    call = _Call(batch, [0.0] * B)
    ref = call.reference(oracle)
    for ticks in (None, -1, 0):
        with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks):
            call()
        got = call.result()
        _equal(got[:2], ref[:2])
        assert not got[2].any()
    assert len(set(ref[1].tolist())) >= 3


# A sequence with a bad temperature leaves its box at once: later calls find it free, the others in the batch are as before.
@pytest.mark.parametrize("B,V,dtype", SIZES)
def test_bad_temperatures_among_good_ones(oracle, B, V, dtype):
    batch, temps = _chain(B, 3, V, dtype, seed=9)
    bad = {1: float("nan"), 6: -1.0, 7: float("inf"), 13: float("-inf"), B - 1: float("nan")}
    call = _Call(batch, temps)
    ref = call.reference(oracle)
    call.temps = torch.tensor([bad.get(b, t) for b, t in enumerate(temps)], dtype=torch.float32, device="cuda")
    good = [b for b in range(B) if b not in bad]
    for _ in range(70):  # (more calls than there are sets of boxes, twice)
        call()
    toks, n, flags = call.result()
    assert (n[list(bad)] == -1).all() and (toks[list(bad)] == -1).all()
    compare_sampler((toks[good], n[good], flags[good]), [r[good] for r in ref])
    call.temps = torch.tensor(temps, dtype=torch.float32, device="cuda")
    call()
    compare_sampler(call.result(), ref)


# Trees of several streams at a time: whatever meets, a call's results have the bits that it has by itself.
def test_trees_of_several_streams():
    trees = [_tree(B, V, "bf16", B, T) for B, V, T in ((128, 131072, 0.6), (64, 151936, 1.0), (100, 100003, 1.3))]
    want = [gpu_tree_sample(tb) for tb in trees]
    streams = [torch.cuda.Stream() for _ in trees]
    torch.cuda.synchronize()
    calls = []
    for tb in trees:
        B, d = len(tb.kv_lens), tb.max_depth
        calls.append([[torch.full(s, -7, dtype=torch.int32, device="cuda") for s in ((B, d + 1), (B, d), (B,), (B,))] for _ in range(20)])
    torch.cuda.synchronize()
    for turn in range(20):
        for tb, outs, s in zip(trees, calls, streams):
            binding.respec_tree_rejection_sample(tb.target_logits, tb.draft_logits, tb.node_tokens, tb.parent, tb.q_indptr, tb.u_accept,
                                                 tb.u_final, *outs[turn], tb.max_rows, tb.max_depth, tb.wl.temperature, stream=s)
    torch.cuda.synchronize()
    for outs, w in zip(calls, want):
        for out in outs:
            _equal([o.cpu().numpy() for o in out], w)
