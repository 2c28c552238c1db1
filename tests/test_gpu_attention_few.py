"""The attention form for few tiles per compute unit against the CPU oracle: the edges of its tiles, of
its parts (a wave without tiles, one part per pair, more pairs of work-groups than parts) and of the rule
that chooses it.  Bounds as everywhere for bf16 attention (test_gpu_attention_forms.py)."""
import numpy as np
import pytest
import torch

from helpers import check_bf16_attention_rows, env_setting, gpu_attention, gpu_tree_attention, oracle_attention, oracle_tree_attention
from paper_2510_26475_amd import binding, synth

pytestmark = pytest.mark.gpu


def _wl(Hq, Hkv, D):
    return synth.Workload("few", B=0, k=0, Hq=Hq, Hkv=Hkv, D=D, V=8, dtype="bf16", len_dist="uniform", len_lo=1, len_hi=1)


def _chain(heads, lens, k, seed):
    ks = [max(0, min(k - (i % 3 == 2), L - 1)) for i, L in enumerate(lens)]
    return synth.make_batch(_wl(*heads), device="cuda", kv_lens=lens, k_per_seq=ks, seed=seed, with_logits=False)


def _check(oracle, batch, sm_scale=None):
    out, lse = gpu_attention(batch, sm_scale=sm_scale)
    ref, ref_lse = oracle_attention(oracle, batch, sm_scale=sm_scale)
    got = out.double().cpu().numpy()
    assert np.isfinite(got).all()
    check_bf16_attention_rows(got, ref)
    assert np.abs(lse.double().cpu().numpy() - ref_lse).max() <= 2e-2


# one to four column tiles at both head sizes; lengths around 16-row halves, tiles and rounds of four waves
@pytest.mark.parametrize("groups", [1, 2])
@pytest.mark.parametrize("heads,k", [((4, 1, 64), 2), ((8, 2, 64), 7), ((16, 2, 64), 5), ((16, 2, 64), 7), ((16, 2, 128), 1),
                                     ((28, 4, 128), 3), ((40, 8, 128), 8), ((28, 4, 128), 8), ((3, 1, 128), 20), ((2, 2, 128), 63)])
@pytest.mark.parametrize("lens", [[64], [65, 79, 80, 81, 96, 97], [128, 129, 160, 257, 4097], [15000, 66, 2049, 500]])
def test_against_the_oracle(oracle, heads, k, lens, groups):
    with env_setting("RESPEC_ATTN_FEW", groups):
        _check(oracle, _chain(heads, lens, k, seed=k + len(lens)))


# as many pairs as work-groups (every sequence one part), a few less, and short caches (the new tokens only)
@pytest.mark.parametrize("heads,B", [((28, 4, 128), 64), ((28, 4, 128), 60), ((40, 8, 128), 32), ((4, 1, 64), 64), ((15, 3, 64), 64)])
def test_many_pairs(oracle, heads, B):
    lens = [1 + (37 * i) % 300 for i in range(B)]
    with env_setting("RESPEC_ATTN_FEW", 1):
        _check(oracle, _chain(heads, lens, 3, seed=B))


# the rule by size, on both sides of its lines in batch size, pairs and tiles
@pytest.mark.parametrize("heads,B,L", [((28, 4, 128), 64, 120), ((28, 4, 128), 65, 120), ((40, 8, 128), 32, 60), ((40, 8, 128), 33, 60),
                                       ((28, 4, 128), 8, 1500), ((28, 4, 128), 16, 4000), ((4, 1, 64), 64, 3000), ((40, 8, 128), 4, 7000)])
@pytest.mark.parametrize("k", [0, 3])
def test_by_size(oracle, heads, B, L, k):
    _check(oracle, _chain(heads, [max(L - 7 * (i % 11), 5) for i in range(B)], k, seed=B + k))


@pytest.mark.parametrize("scale", [-0.2, 0.0, 3.0])
def test_scales(oracle, scale):
    with env_setting("RESPEC_ATTN_FEW", 1):
        _check(oracle, _chain((16, 2, 128), [700, 5, 97], 4, seed=5), sm_scale=scale)


# a reference that moves at nearly every tile, and one that never moves after the first
@pytest.mark.parametrize("falling", [False, True])
def test_moving_references(oracle, falling):
    batch = _chain((28, 4, 128), [2100, 333], 3, seed=9)
    ramp = torch.cat([torch.linspace(0.2, 6.0, L) for L in (2100, 333)]).to("cuda")
    ramp = ramp.flip(0) if falling else ramp
    batch.k_cache.copy_((batch.k_cache.float().abs() * 0.05 + ramp[:, None, None]).to(torch.bfloat16))
    batch.q.copy_(batch.q.float().abs().to(torch.bfloat16))
    with env_setting("RESPEC_ATTN_FEW", 2):
        _check(oracle, batch)


# trees, contiguous and paged (halves of a tile in two pages), and the later layers of a forward
@pytest.mark.parametrize("heads", [(28, 4, 128), (8, 2, 64)])
@pytest.mark.parametrize("page_size", [16, 64])
def test_trees_pages_and_layers(oracle, heads, page_size):
    parents = [synth.caterpillar_parents(2, 2)] * 5
    lens = [40, 777, 5, 100, 1500]
    batch = synth.make_tree_batch(_wl(*heads), parents, device="cuda", kv_lens=lens, seed=3, with_logits=False)
    scale = 1.0 / np.sqrt(heads[2])
    paged = synth.paginate(batch.k_cache, batch.v_cache, batch.kv_lens, page_size, seed=1)
    with env_setting("RESPEC_ATTN_FEW", 1):
        out, lse = gpu_tree_attention(batch)
        ref, ref_lse = oracle_tree_attention(oracle, batch)
        check_bf16_attention_rows(out.double().cpu().numpy(), ref)
        assert np.abs(lse.double().cpu().numpy() - ref_lse).max() <= 2e-2
        ws = torch.empty(binding.respec_verify_attention_workspace_bytes(
            5, batch.total_q, paged.num_pages * page_size, batch.max_rows, batch.max_kv_len, *heads, binding.RESPEC_BF16),
            dtype=torch.uint8, device="cuda")
        for call in (binding.respec_verify_attention_paged, binding.respec_verify_attention_paged_next_layer):
            again = torch.full_like(batch.q, float("nan"))
            call(batch.q, paged.k_pages, paged.v_pages, batch.q_indptr, paged.page_indptr, paged.page_table, paged.kv_len, again,
                 None, batch.max_rows, batch.max_kv_len, scale, ws, tree_mask=batch.tree_mask)
            torch.cuda.synchronize()
            assert torch.equal(out, again)
