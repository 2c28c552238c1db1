"""The combine kernel's forms (waves that share a column's parts) against the CPU oracle.

Partials carry 2^-16 of a row's largest magnitude and the fold runs in fp32, so the bounds are the
attention's own: 2e-2 absolute, and 2^-7 of the row's largest magnitude plus 1e-3 per element.
"""
import math

import numpy as np
import pytest

from helpers import attn_wgs, check_bf16_attention_rows, env_setting, gpu_attention, oracle_attention
from paper_2510_26475_amd import synth

pytestmark = pytest.mark.gpu


# few tiles and many parts (most parts own none), one long sequence among short ones, one sequence
# cut into 64 or more parts, a row count that leaves the last column group ragged
@pytest.mark.parametrize("form", [1, 4, 8])
@pytest.mark.parametrize("wgs", [None, 3, 64, 1024])
@pytest.mark.parametrize("shape", [(28, 4, 128, [4097], [2]), (16, 2, 128, [33, 70, 6000, 9], [4, 0, 3, 4]),
                                   (4, 1, 64, [40, 3000, 5], [6, 1, 4]), (40, 8, 128, [1, 65, 640], [0, 8, 2])])
def test_combine_forms_agree_with_the_oracle(oracle, shape, wgs, form):
    Hq, Hkv, D, lens, ks = shape
    wl = synth.Workload("combine", B=0, k=0, Hq=Hq, Hkv=Hkv, D=D, V=8, dtype="bf16", len_dist="uniform", len_lo=1, len_hi=1)
    batch = synth.make_batch(wl, device="cuda", kv_lens=lens, k_per_seq=ks, seed=Hq + form, with_logits=False)
    with env_setting("RESPEC_ATTN_COMBINE", form), attn_wgs(wgs):
        out, lse = gpu_attention(batch)
    ref, ref_lse = oracle_attention(oracle, batch)
    got = out.double().cpu().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 2e-2
    check_bf16_attention_rows(got, ref, 2.5e-3)
    # fp32 sums of up to 6000 terms of bf16 products: a few 1e-6 in the logarithm
    assert np.abs(lse.double().cpu().numpy() - ref_lse).max() <= 1e-4 * max(1.0, math.log(max(lens)))
