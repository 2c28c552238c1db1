"""Sequences shared between work-groups without a workspace (one temperature per sequence, trees of drafts):
the parts meet in the library's own mailboxes, or part 0 walks alone.  Exact against the CPU oracle on
unflagged sequences either way, in order, beside other calls and under replay."""
import numpy as np
import pytest
import torch

from helpers import compare_sampler, compare_tree_sampler, env_setting, gpu_tree_sample, oracle_tree_sample
from paper_2510_26475_amd import binding, synth

pytestmark = pytest.mark.gpu

TEMPS = (0.6, 0.0, 1.0, 0.4)


def _wl(B, k, V, dtype, T=0.6):
    return synth.Workload("claim", B=B, k=k, Hq=8, Hkv=1, D=64, V=V, dtype=dtype, len_dist="uniform", len_lo=64, len_hi=64, temperature=T)


def _chain(B, k, V, dtype, seed):
    batch = synth.make_batch(_wl(B, k, V, dtype), device="cuda", kv_lens=[64] * B, k_per_seq=[(k, k, 1, 0)[b % 4] for b in range(B)], seed=seed,
                             with_attention=False)
    return batch, [TEMPS[(b * 7 + b // 4) % 4] for b in range(B)]


class _Call:
    """A call with one temperature per sequence and buffers of its own."""

    def __init__(self, batch, temps):
        B, dev = len(batch.k_per_seq), "cuda"
        self.batch, self.temps = batch, torch.tensor(temps, dtype=torch.float32, device=dev)
        self.toks = torch.full((B, batch.max_k + 1), -7, dtype=torch.int32, device=dev)
        self.n, self.flags = (torch.full((B,), -7, dtype=torch.int32, device=dev) for _ in range(2))

    def __call__(self):
        b = self.batch
        binding.respec_rejection_sample_per_seq(b.target_logits, b.draft_logits, b.draft_tokens, b.q_indptr, b.u_accept, b.u_final,
                                                self.temps, self.toks, self.n, self.flags, b.max_k)

    def result(self):
        torch.cuda.synchronize()
        return self.toks.cpu().numpy(), self.n.cpu().numpy(), self.flags.cpu().numpy()

    def reference(self, oracle):
        b = self.batch
        dt = oracle.F32 if b.wl.dtype == "f32" else oracle.BF16
        return oracle.rejection_sample_per_seq(
            synth.to_host_array(b.target_logits), synth.to_host_array(b.draft_logits), b.draft_tokens.cpu().numpy(),
            b.q_indptr.cpu().numpy(), b.u_accept.cpu().numpy(), b.u_final.cpu().numpy(), b.max_k, self.temps.cpu().numpy(), dt,
            n_threads=0)


def _tree(B, V, dtype, seed, T):
    shapes = [synth.caterpillar_parents(3, 2), synth.caterpillar_parents(2, 4), [-1], [-1, 0, 1, 2]]
    return synth.make_tree_batch(_wl(B, 6, V, dtype, T), [shapes[b % 4] for b in range(B)], device="cuda", kv_lens=[64] * B, seed=seed,
                                 with_attention=False)


# parts of two and four, one and two items per stage, whole and ragged rows; ticks 0: whoever does not find the others
# at once gives up, so sequences are walked alone, shared, or found given up; ticks -1: all are walked alone
@pytest.mark.parametrize("ticks", [None, 0, -1])
@pytest.mark.parametrize("B,V,dtype", [(1, 151936, "bf16"), (9, 151936, "bf16"), (64, 33000, "bf16"), (65, 52000, "bf16"), (128, 65536, "bf16"),
                                       (20, 77777, "bf16"), (33, 50257, "f32"), (70, 80001, "f32"), (5, 151936, "f32")])
def test_temperatures(oracle, B, V, dtype, ticks):
    batch, temps = _chain(B, 4, V, dtype, seed=B)
    call = _Call(batch, temps)
    ref = call.reference(oracle)
    with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks):
        for _ in range(3):
            call()
            compare_sampler(call.result(), ref)


@pytest.mark.parametrize("ticks", [None, 0, -1])
@pytest.mark.parametrize("B,V,dtype,T", [(1, 151936, "bf16", 0.6), (9, 151936, "bf16", 1.0), (64, 131072, "bf16", 0.6), (70, 100003, "bf16", 1.0),
                                         (20, 77777, "bf16", 0.6), (12, 80001, "f32", 0.6), (5, 151936, "f32", 1.0)])
def test_trees(oracle, B, V, dtype, T, ticks):
    tb = _tree(B, V, dtype, B, T)
    ref = oracle_tree_sample(oracle, tb)
    with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks):
        for _ in range(3):
            compare_tree_sampler(gpu_tree_sample(tb), ref)


# a forced split that leaves the last parts of a short row without a slot, greedy sequences among the others; the last row ends
# with its buffer
@pytest.mark.parametrize("ticks", [None, -1])
@pytest.mark.parametrize("V,dtype", [(1024, "bf16"), (512, "f32"), (520, "bf16"), (64, "bf16"), (32, "f32")])
def test_parts_without_slots(oracle, V, dtype, ticks):
    batch, temps = _chain(12, 3, V, dtype, seed=V)
    first = batch.target_logits[0].float().argmax().int()
    batch.draft_tokens[0] = first  # a greedy sequence that goes on past its first draft
    call = _Call(batch, [0.0] * 4 + temps[4:])
    with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks), env_setting("RESPEC_SAMPLER_SPLIT", 4):
        call()
        ref = call.reference(oracle)
        compare_sampler(call.result(), ref)
        assert ref[1][0] >= 1


# what the interface says is never read may hold anything: a root's token and uniform, a greedy sequence's uniforms and drafter rows
@pytest.mark.parametrize("V", [151936, 2048, 2047])
def test_entries_that_are_not_used(oracle, V):
    tb = _tree(32, V, "bf16", 3, 0.6)
    want = gpu_tree_sample(tb)
    root = tb.q_indptr[:-1].long()
    tb.u_accept[root] = float("nan")
    tb.node_tokens[root] = 0x7fffffff
    for a, b in zip(want, gpu_tree_sample(tb)):
        np.testing.assert_array_equal(a, b)
    batch, temps = _chain(32, 3, V, "bf16", seed=4)
    call = _Call(batch, temps)
    call()
    want = [a.copy() for a in call.result()]
    for b, (k, q0) in enumerate(zip(batch.k_per_seq, batch.q_indptr.tolist())):
        if temps[b] == 0.0:
            batch.u_final[b] = float("nan")
            batch.u_accept[q0 - b:q0 - b + k] = float("nan")
            batch.draft_logits[q0 - b:q0 - b + k] = float("nan")
    call()
    for a, b in zip(want, call.result()):
        np.testing.assert_array_equal(a, b)


def _edge_uniforms(weights, count):
    """Binary32 uniforms on top of edges of a distribution's cells, where the last bits of the sums decide the token."""
    cdf = weights.double().cumsum(0)
    cdf = cdf / cdf[-1]
    cdf = cdf[(cdf > 0.25) & (cdf < 0.999999)]
    near = (cdf.float().double() - cdf).abs().argsort()[:count]
    return cdf[near].float()


def _on_edges(target, draft, k, T):
    """Draft tokens that are rejected (uniform 0.999) and final uniforms on edges of what is then drawn from: the residual,
    or the target row where there is no draft."""
    p, q = torch.softmax(target.double() / T, -1), torch.softmax(draft.double() / T, -1)
    x = (q - p).argmax(-1)
    ratio = (p / q).gather(1, x[:, None])
    assert bool((ratio < 0.99).all())
    w = torch.where(torch.tensor(k, device=p.device)[:, None] > 0, (p - q).clamp_min(0), p)
    return x.int(), torch.cat([_edge_uniforms(w[b], 8)[b % 8, None] for b in range(len(k))])


# The bits of a sequence's sums, and so its tokens on the edges of cells, do not depend on whether its parts met.
@pytest.mark.parametrize("kind", ["temperatures", "tree"])
@pytest.mark.parametrize("B,V,dtype,T", [(64, 151936, "bf16", 1.0), (128, 151936, "bf16", 0.6), (48, 80001, "f32", 0.6), (50, 100003, "bf16", 1.3)])
def test_meeting_does_not_change_a_result(kind, B, V, dtype, T):
    k = [b % 2 for b in range(B)]
    if kind == "tree":
        batch = synth.make_tree_batch(_wl(B, 1, V, dtype, T), [[-1] + [0] * n for n in k], device="cuda", kv_lens=[64] * B, seed=7, with_attention=False)
        rows = batch.q_indptr[:-1].long()
        x, batch.u_final[:] = _on_edges(batch.target_logits[rows], batch.draft_logits[rows], k, T)
        child = rows[1::2] + 1
        batch.node_tokens[child] = x[1::2]
        batch.u_accept[child] = 0.999
        call = lambda: gpu_tree_sample(batch)  # noqa: E731
    else:
        batch = synth.make_batch(_wl(B, 1, V, dtype, T), device="cuda", kv_lens=[64] * B, k_per_seq=k, seed=7, with_attention=False)
        rows = batch.q_indptr[:-1].long()
        draft = batch.draft_logits.repeat_interleave(2, 0)  # (of sequences without a draft nothing is used)
        x, batch.u_final[:] = _on_edges(batch.target_logits[rows], draft, k, T)
        batch.draft_tokens[:] = x[1::2]
        batch.u_accept[:] = 0.999
        one = _Call(batch, [T] * B)

        def call():
            one()
            return one.result()
    first = None
    for ticks in (None, -1, 0, 0, 0, None):
        with env_setting("RESPEC_SAMPLER_CLAIM_TICKS", ticks):
            got = [a.copy() for a in call()]
        first = first or got
        for a, b in zip(first, got):
            np.testing.assert_array_equal(a, b)
    assert (first[-2] == 0).all() and (first[-1] & 2).sum() > B // 2  # drafts rejected, draws on edges


# calls of several streams at a time (their work-groups compete for the compute units), and replays of a graph
def test_streams_and_replays(oracle):
    calls = []
    for i, B in enumerate((100, 60, 128)):
        batch, temps = _chain(B, 3, 65536, "bf16", seed=20 + i)
        calls.append(_Call(batch, temps))
        calls[-1]()
    torch.cuda.synchronize()
    refs = [c.reference(oracle) for c in calls]
    streams = [torch.cuda.Stream() for _ in calls]
    for _ in range(40):
        for c, s in zip(calls, streams):
            with torch.cuda.stream(s):
                c()
    for c, ref in zip(calls, refs):
        compare_sampler(c.result(), ref)
    between = _Call(calls[0].batch, calls[0].temps.tolist())  # (buffers of its own: what a replay wrote is looked at)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for c in calls:
            c()
    for _ in range(3):
        for c in calls + [between]:
            c.toks.zero_()
            c.n.fill_(-7)
        graph.replay()
        between()  # eager work between the replays
        for c, ref in zip(calls + [between], refs + refs[:1]):
            compare_sampler(c.result(), ref)
