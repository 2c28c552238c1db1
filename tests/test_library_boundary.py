"""CPU-side checks of the C boundary: the library loads, exports every symbol the header
declares, and rejects bad arguments on the host before anything touches a GPU."""
import ctypes
import os
import re

import pytest

from paper_2510_26475_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(build.LIB_PATH):
        build.build()
    return binding.load()


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "respec.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(respec_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared_symbols()
    assert set(names) == set(binding.EXPORTED_SYMBOLS)
    for name in names:
        assert getattr(lib, name) is not None


def test_version_and_status_strings(lib):
    assert lib.respec_version() >= 100
    texts = {lib.respec_status_string(i).decode() for i in range(5)}
    assert len(texts) == 5 and "ok" in texts


def test_workspace_query(lib):
    f = lib.respec_verify_attention_workspace_bytes
    a = f(256, 1024, 668000, 4, 8192, 28, 4, 128, binding.RESPEC_BF16)
    assert a > 0 and a % 256 == 0
    assert f(256, 1024, 668000, 4, 8192, 28, 5, 128, binding.RESPEC_BF16) == 0     # Hq % Hkv
    assert f(256, 1024, 668000, 4, 8192, 28, 4, 96, binding.RESPEC_BF16) == 0      # head size
    assert f(0, 0, 0, 4, 8192, 28, 4, 128, binding.RESPEC_BF16) == 0
    w = lib.respec_rejection_sample_workspace_bytes(256, 1024, 151936, binding.RESPEC_BF16)
    assert w > 0 and w % 256 == 0                  # one mailbox per sequence
    assert lib.respec_rejection_sample_workspace_bytes(0, 0, 151936, binding.RESPEC_BF16) == 0


def test_a_distillation_workspace_is_enough_for_fewer_rows(lib):
    # (fewer rows are shared by more work-groups: a call with a buffer sized for the largest one must not lose its form)
    size = lib.respec_kd_rows_workspace_bytes
    for dt, epv in ((binding.RESPEC_BF16, 8), (binding.RESPEC_F32, 4)):
        for V in (epv, 8000, 16000, 20480, 32000, 50256, 96000, 128000, 151936, 400000, 32 * 2432 * epv, 32 * 2432 * epv + epv):
            sizes = [size(rows, V, dt) for rows in list(range(1, 600)) + [1023, 1024, 2047, 2048, 4096]]
            assert all(s % 256 == 0 and s >= 8 for s in sizes) and sizes == sorted(sizes), (V, dt)


def test_distillation_rows_are_shared_only_where_that_is_no_slower(lib):
    # the size tells: 8 bytes a row where it is streamed, 72 bytes a row and member where a team keeps it (a size is also enough
    # for fewer rows, which rows of 48,000 logits and more are shared for)
    size = lib.respec_kd_rows_workspace_bytes
    bf16, f32 = binding.RESPEC_BF16, binding.RESPEC_F32
    for rows, V, dt in [(64, 32000, bf16), (32, 40000, bf16), (64, 40000, f32), (2047, 32000, bf16), (1024, 11200, f32), (2048, 40000, bf16),
                        (2048, 20000, f32)]:                               # (were slower by 4 to 20 %, 2047 rows aside)
        assert size(rows, V, dt) == (8 * rows + 255) // 256 * 256, (rows, V, dt)
    for rows, V, dt in [(256, 96000, bf16), (2048, 48000, bf16), (2048, 80000, bf16)]:
        assert size(rows, V, dt) < 288 * rows, (rows, V, dt)
    for rows, V, dt, team in [(8, 151936, bf16, 32), (64, 48000, f32, 8), (2048, 32000, bf16, 2), (2048, 64000, bf16, 4), (2048, 32000, f32, 4),
                              (256, 151936, bf16, 8), (1500, 11200, f32, 2)]:
        assert 72 * rows * team <= size(rows, V, dt) <= 72 * rows * team + 512, (rows, V, dt)


def test_attention_argument_errors_need_no_gpu(lib):
    null = ctypes.c_void_p(None)
    bogus = ctypes.c_void_p(0x1000)
    call = lib.respec_verify_attention
    # null pointers
    st = call(null, null, null, null, null, null, null, 1, 4, 100, 4, 100, 8, 2, 128, 0.1,
              binding.RESPEC_BF16, null, 0, null)
    assert st == 1 and b"null" in lib.respec_last_error()
    # Hq not a multiple of Hkv
    st = call(bogus, bogus, bogus, bogus, bogus, bogus, null, 1, 4, 100, 4, 100, 7, 2, 128, 0.1,
              binding.RESPEC_BF16, bogus, 1 << 30, null)
    assert st == 1
    # unsupported head size
    st = call(bogus, bogus, bogus, bogus, bogus, bogus, null, 1, 4, 100, 4, 100, 8, 2, 96, 0.1,
              binding.RESPEC_BF16, bogus, 1 << 30, null)
    assert st == 2
    # cache shorter than the new tokens
    st = call(bogus, bogus, bogus, bogus, bogus, bogus, null, 1, 4, 3, 4, 3, 8, 2, 128, 0.1,
              binding.RESPEC_BF16, bogus, 1 << 30, null)
    assert st == 1
    # misaligned q
    st = call(ctypes.c_void_p(0x1004), bogus, bogus, bogus, bogus, bogus, null, 1, 4, 100, 4, 100,
              8, 2, 128, 0.1, binding.RESPEC_BF16, bogus, 1 << 30, null)
    assert st == 1 and b"aligned" in lib.respec_last_error()
    # workspace too small
    st = call(bogus, bogus, bogus, bogus, bogus, bogus, null, 1, 4, 100, 4, 100, 8, 2, 128, 0.1,
              binding.RESPEC_BF16, bogus, 16, null)
    assert st == 3


def test_sampler_argument_errors_need_no_gpu(lib):
    null = ctypes.c_void_p(None)
    bogus = ctypes.c_void_p(0x1000)
    call = lib.respec_rejection_sample

    def run(**kw):
        a = dict(t=bogus, d=bogus, tok=bogus, qi=bogus, ua=bogus, uf=bogus, ot=bogus, on=bogus,
                 of=null, B=2, total_q=8, max_k=3, V=1024, ld_t=1024, ld_d=1024, T=1.0,
                 dt=binding.RESPEC_F32)
        a.update(kw)
        return call(a["t"], a["d"], a["tok"], a["qi"], a["ua"], a["uf"], a["ot"], a["on"], a["of"],
                    a["B"], a["total_q"], a["max_k"], a["V"], a["ld_t"], a["ld_d"], a["T"], a["dt"],
                    null, 0, null)

    assert run(T=0.0) == 1
    assert run(T=-1.0) == 1
    assert run(T=float("nan")) == 1
    assert run(t=null) == 1
    assert run(d=null) == 1                  # drafts present but no drafter logits
    assert run(ld_t=1000) == 1               # stride below V
    assert run(max_k=2) == 1                 # 2 sequences * 2 < 6 drafted tokens
    assert run(V=0) == 1
    assert run(dt=7) == 1
    assert run(B=0) == 1


def test_tree_entry_points_argument_errors_need_no_gpu(lib):
    null = ctypes.c_void_p(None)
    bogus = ctypes.c_void_p(0x1000)
    attn = lib.respec_verify_attention_tree
    # more rows per sequence than the mask has bits
    st = attn(bogus, bogus, bogus, bogus, bogus, bogus, bogus, null, 1, 65, 100, 65, 100, 8, 2, 128, 0.1,
              binding.RESPEC_BF16, bogus, 1 << 30, null)
    assert st == 2
    # no mask
    st = attn(bogus, bogus, bogus, bogus, bogus, null, bogus, null, 1, 4, 100, 4, 100, 8, 2, 128, 0.1,
              binding.RESPEC_BF16, bogus, 1 << 30, null)
    assert st == 1
    call = lib.respec_tree_rejection_sample

    def run(**kw):
        a = dict(t=bogus, d=bogus, tok=bogus, par=bogus, qi=bogus, ua=bogus, uf=bogus, ot=bogus, op=bogus,
                 on=bogus, of=null, B=2, total_q=8, max_rows=4, max_depth=3, V=1024, ld_t=1024, ld_d=1024,
                 T=1.0, dt=binding.RESPEC_F32)
        a.update(kw)
        return call(a["t"], a["d"], a["tok"], a["par"], a["qi"], a["ua"], a["uf"], a["ot"], a["op"], a["on"],
                    a["of"], a["B"], a["total_q"], a["max_rows"], a["max_depth"], a["V"], a["ld_t"], a["ld_d"],
                    a["T"], a["dt"], null)

    assert run(T=0.0) == 1
    assert run(T=float("inf")) == 1
    assert run(d=null) == 1
    assert run(par=null) == 1
    assert run(op=null) == 1
    assert run(ld_d=1000) == 1
    assert run(max_rows=3) == 1              # 2 sequences * 3 rows < 8 rows
    assert run(max_rows=65, total_q=100) == 2
    assert run(max_depth=-1) == 1
    assert run(dt=7) == 1


def test_the_current_stream_is_found_without_torchs_private_function(monkeypatch):
    import torch
    from types import SimpleNamespace
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=41))
    monkeypatch.setattr(binding, "_current_raw_stream", lambda device: 100 + device)
    assert binding._stream_ptr(None) == 103
    assert binding._stream_ptr(SimpleNamespace(cuda_stream=7)) == 7
    monkeypatch.setattr(binding, "_current_raw_stream", None)
    assert binding._stream_ptr(None) == 41
