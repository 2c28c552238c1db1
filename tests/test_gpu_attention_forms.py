"""The attention kernel's forms (consumers per range and per work-group) against the CPU oracle.

Each form is forced, so that small batches reach the ones that the sizes alone would not choose.
Bounds as everywhere for bf16 attention: 2e-2 absolute, 2^-7 of the row's largest magnitude plus
1e-3 per element (one rounding of the probabilities, one of the output).
"""
import contextlib

import numpy as np
import pytest
import torch

from helpers import attn_wgs, check_bf16_attention_rows, env_setting, gpu_attention, oracle_attention
from paper_2510_26475_amd import binding, synth

pytestmark = pytest.mark.gpu

# (knobs, what they force)
FORMS = {
    "four per range, eight per work-group": {"RESPEC_ATTN_QUAD": 2, "RESPEC_ATTN_CONSUMERS": 8},
    "four per range, four per work-group": {"RESPEC_ATTN_QUAD": 2, "RESPEC_ATTN_CONSUMERS": 4},
    "two per range, eight per work-group": {"RESPEC_ATTN_QUAD": 0, "RESPEC_ATTN_WIDE": 1},
    "by size": {},
}


@contextlib.contextmanager
def _form(name):
    with contextlib.ExitStack() as stack:
        for k, v in FORMS[name].items():
            stack.enter_context(env_setting(k, v))
        yield


def _wl(Hq, Hkv, D):
    return synth.Workload("forms", B=0, k=0, Hq=Hq, Hkv=Hkv, D=D, V=8, dtype="bf16", len_dist="uniform", len_lo=1, len_hi=1)


def _check(oracle, batch, sm_scale=None):
    out, lse = gpu_attention(batch, sm_scale=sm_scale)
    ref, ref_lse = oracle_attention(oracle, batch, sm_scale=sm_scale)
    got = out.double().cpu().numpy()
    assert np.isfinite(got).all()
    check_bf16_attention_rows(got, ref)
    assert np.abs(lse.double().cpu().numpy() - ref_lse).max() <= 2e-2
    return out


# 17, 28, 33, 45, 64 and (blocks of 128, the last consumers without columns) 72, 91, 128, 136 columns
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("wgs", [None, 1, 5, 512])
@pytest.mark.parametrize("shape", [(17, 1, 128, 0), (28, 4, 128, 3), (11, 1, 128, 2), (40, 8, 128, 8), (16, 2, 64, 7),
                                   (16, 2, 128, 8), (28, 4, 128, 12), (8, 1, 64, 15), (16, 2, 128, 16)])
def test_forms_agree_with_the_oracle(oracle, shape, wgs, form):
    Hq, Hkv, D, k = shape
    lens = [33, 700, k + 1, 31 + k, 32 + k, 64, 2049, 97]
    ks = [k, k, k, max(k - 1, 0), k, 0, k, min(k, 3)]
    lens = [max(L, kk + 1) for L, kk in zip(lens, ks)]
    batch = synth.make_batch(_wl(Hq, Hkv, D), device="cuda", kv_lens=lens, k_per_seq=ks, seed=Hq + k, with_logits=False)
    with _form(form), attn_wgs(wgs):
        _check(oracle, batch)


# Few sequences that share all ranges: the main kernel on both sides of its line (two tiles per consumer of the device) and
# well beyond it, and the form for few tiles, which takes the same batches by size
@pytest.mark.usefixtures("attn_few")
@pytest.mark.parametrize("pairs,tiles", [(1, 1), (1, 2), (1, 3), (4, 2), (4, 3), (4, 4), (16, 3), (18, 2)])
def test_few_long_sequences(oracle, pairs, tiles):
    B, Hkv = {1: (1, 1), 4: (2, 2), 16: (8, 2), 18: (9, 2)}[pairs]
    consumers = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    lens = [(2 * tiles + 1) * consumers * 16 // pairs - 3 * i for i in range(B)]
    batch = synth.make_batch(_wl(8 * Hkv, Hkv, 64), device="cuda", kv_lens=lens, k_per_seq=[2] * B, seed=pairs + tiles, with_logits=False)
    _check(oracle, batch)


# The scale is folded into the exponent: its sign, a value of zero (uniform attention over the
# visible keys), large ones (one key dominates, references move often) and tiny ones
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("scale", [-0.2, 0.0, 1e-30, -3.0, 3.0])
def test_scales(oracle, form, scale):
    batch = synth.make_batch(_wl(16, 2, 128), device="cuda", kv_lens=[300, 5, 97], k_per_seq=[4, 4, 2], seed=5, with_logits=False)
    with _form(form):
        _check(oracle, batch, sm_scale=scale)


# scores that grow along the sequence, so that a reference moves at nearly every tile, and scores
# whose first tile dominates, so that it never moves again
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("falling", [False, True])
def test_moving_references(oracle, form, falling):
    batch = synth.make_batch(_wl(28, 4, 128), device="cuda", kv_lens=[900, 333], k_per_seq=[3, 2], seed=9, with_logits=False)
    ramp = torch.cat([torch.linspace(0.2, 6.0, L) for L in (900, 333)]).to("cuda")
    ramp = ramp.flip(0) if falling else ramp
    batch.k_cache.copy_((batch.k_cache.float().abs() * 0.05 + ramp[:, None, None]).to(torch.bfloat16))
    batch.q.copy_(batch.q.float().abs().to(torch.bfloat16))
    with _form(form):
        _check(oracle, batch)


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("page_size", [16, 64])
def test_paged_and_trees_are_bit_equal_to_contiguous(form, page_size):
    wl = _wl(28, 4, 128)
    parents = [synth.caterpillar_parents(2, 2)] * 5
    batch = synth.make_tree_batch(wl, parents, device="cuda", kv_lens=[40, 777, 5, 100, 1500], seed=3, with_logits=False)
    paged = synth.paginate(batch.k_cache, batch.v_cache, batch.kv_lens, page_size, seed=1)
    outs = []
    with _form(form), attn_wgs(24):
        for use_pages in (False, True):
            out = torch.full_like(batch.q, float("nan"))
            total = paged.num_pages * page_size if use_pages else batch.total_kv
            ws = torch.empty(binding.respec_verify_attention_workspace_bytes(
                5, batch.total_q, total, batch.max_rows, batch.max_kv_len, 28, 4, 128, binding.RESPEC_BF16),
                dtype=torch.uint8, device="cuda")
            if use_pages:
                binding.respec_verify_attention_paged(batch.q, paged.k_pages, paged.v_pages, batch.q_indptr, paged.page_indptr,
                                                      paged.page_table, paged.kv_len, out, None, batch.max_rows,
                                                      batch.max_kv_len, 0.088, ws, tree_mask=batch.tree_mask)
            else:
                binding.respec_verify_attention_tree(batch.q, batch.k_cache, batch.v_cache, batch.q_indptr, batch.kv_indptr,
                                                     batch.tree_mask, out, None, batch.max_rows, batch.max_kv_len, 0.088, ws)
            torch.cuda.synchronize()
            outs.append(out)
    assert torch.isfinite(outs[0].float()).all()
    assert torch.equal(outs[0], outs[1])


# A caller without a bound on the lengths passes the largest int32: the same split, the same bits (the
# combine kernel's form follows the bound and is held)
@pytest.mark.usefixtures("attn_few")
def test_no_bound_on_the_lengths(oracle):
    batch = synth.make_batch(_wl(28, 4, 128), device="cuda", kv_lens=[4096, 3000, 4095, 31, 2048, 4000, 4096, 3500],
                             k_per_seq=[0] * 8, seed=4, with_logits=False)
    outs = []
    with env_setting("RESPEC_ATTN_COMBINE", 1):
        for bound in (4096, 2 ** 31 - 1):
            out = torch.full_like(batch.q, float("nan"))
            ws = torch.empty(binding.respec_verify_attention_workspace_bytes(
                8, batch.total_q, batch.total_kv, 1, bound, 28, 4, 128, binding.RESPEC_BF16), dtype=torch.uint8, device="cuda")
            binding.respec_verify_attention(batch.q, batch.k_cache, batch.v_cache, batch.q_indptr, batch.kv_indptr, out, None,
                                            1, bound, 0.088, ws)
            torch.cuda.synchronize()
            outs.append(out)
    assert torch.isfinite(outs[0].float()).all()
    assert torch.equal(outs[0], outs[1])
