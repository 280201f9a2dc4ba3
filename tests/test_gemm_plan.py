"""Host-only checks of the kernel choice of the bf16 products (alr_debug_gemm_plan), which the GPU
tests use to show that a case reaches the path it is there for."""
import dataclasses

import pytest

from paper_2609_38795_amd import binding, workloads as W

RING128X64, LDS128, WIDE, LDS64 = 2, 4, 5, 6


def _plan(shape, site, rows, cols=0, tokens=8192, anchors=1024, n_cu=256):
    return binding.gemm_plan(shape, binding.make_limits(tokens, 8, anchors, 16), site, rows, cols,
                             n_cu)


def test_headline_choices():
    s = W.get("llama8b_like").shape
    for site in ("prefill_qkv", "prefill_o", "prefill_gu", "prefill_down"):
        assert _plan(s, site, 32768, tokens=32768) == (WIDE, 1, 1), site
    assert _plan(s, "decode_qkv", 1024)[:2] == (WIDE, 2)
    assert _plan(s, "decode_gu", 1024) == (WIDE, 1, 1)
    assert _plan(s, "lm_gemm", 1024)[1:] == (1, 1)


def test_slices_need_their_scratch():
    """8 slices of few rows fit the split-K buffer; rows beyond what it was sized for are not cut."""
    s = dataclasses.replace(W.get("small_bf16").shape, d_model=2048)
    assert _plan(s, "decode_qkv", 8, anchors=8)[1] == 8
    assert _plan(s, "prefill_qkv", 256, anchors=1)[1] == 1


def test_sliced_last_round_depends_on_the_device():
    """7B-like down projection of 10,900 rows: 602 tiles leave 90 of a third round on 256 CUs, and none
    on 301."""
    s = W.get("vl_prefix_7b").shape
    assert _plan(s, "prefill_down", 10900, tokens=10900) == (WIDE, 1, 2)
    assert _plan(s, "prefill_down", 10900, tokens=10900, n_cu=301) == (WIDE, 1, 1)


def test_where_64x128_tiles_are_taken():
    """1B-like prefill: above 128 rows while larger tiles leave CUs idle and the weights are small; not
    for the 33 MB of an 8B-like layer's O."""
    s = W.get("small_bf16").shape
    plan = lambda rows, shape=s, site="prefill_qkv": _plan(shape, site, rows, anchors=1)[0]
    assert plan(128) != LDS64 and plan(300) == LDS64 and plan(600) == LDS64
    assert plan(2048) == LDS128 and plan(32768) == WIDE
    assert plan(2048, site="prefill_o") == LDS64  # 256 tiles of K = 1024
    assert plan(300, W.get("llama8b_like").shape, "prefill_o") == RING128X64


@pytest.mark.parametrize("d_model,rows,kernel", [
    (256, 2830, LDS64), (512, 3072, LDS64),  # a round of 138 and 216 tiles of 128x128 would do
    (576, 3072, LDS128)])
def test_short_k_with_an_epilogue_takes_64x128_tiles(d_model, rows, kernel):
    s = dataclasses.replace(W.get("small_bf16").shape, d_model=d_model, n_heads=4, n_kv_heads=4,
                            head_dim=96 if d_model > 256 else 64)
    assert _plan(s, "prefill_qkv", rows, anchors=1) == (kernel, 1, 1)


@pytest.mark.parametrize("d_model,rows,kernel", [
    (512, 256, RING128X64), (512, 257, LDS64), (640, 700, LDS64), (256, 511, RING128X64),
    (256, 512, LDS64), (576, 300, RING128X64)])
def test_short_k_of_some_hundred_rows(d_model, rows, kernel):
    """Gate/up of 512 columns: 64x128 tiles from 128 K elements of A on, where K is whole 128s."""
    s = dataclasses.replace(W.get("small_bf16").shape, d_model=d_model, d_ffn=256)
    assert _plan(s, "prefill_gu", rows, anchors=1) == (kernel, 1, 1)


def test_plan_errors():
    s = W.get("small_bf16").shape
    for bad in (dict(site="prefill_attn"), dict(rows=0), dict(cols=32), dict(n_cu=0)):
        with pytest.raises(binding.AlrError) as e:
            _plan(s, **{"site": "decode_o", "rows": 4, **bad})
        assert e.value.status == 1, bad
    with pytest.raises(binding.AlrError) as e:
        _plan(W.get("tiny_fp32").shape, "decode_o", 4)
    assert e.value.status == 5
