"""GPU parity: the HIP path through the C ABI against the CPU oracle on the same seeded inputs."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2609_38795_amd import binding, workloads as W
from parity import compare
from gpu_util import make_engine, n_cu, prefill, runner

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _print(*a):
    print(*a, flush=True)


# ------------------------------------------------------------------ GEMM kernels
@pytest.mark.parametrize("dtype,tile", [("bf16", 0), ("f32", 0), ("bf16", 1), ("bf16", 2),
                                        ("bf16", 3), ("bf16", 4), ("bf16", 5), ("bf16", 17),
                                        ("bf16", 18), ("bf16", 19), ("bf16", 20)])
@pytest.mark.parametrize("M,N,K", [(1, 64, 64), (300, 192, 256), (1024, 640, 1152),
                                   (257, 320, 1536)])
def test_gemm_kernel(dtype, tile, M, N, K):
    """Every GEMM kernel variant against a float64 product, ragged M and partial N tiles."""
    _print(f"gemm {dtype} tile {tile} {M}x{N}x{K}")
    rng = np.random.default_rng(M + N + K)
    a = rng.standard_normal((M, K)).astype(np.float32)
    w = rng.standard_normal((N, K)).astype(np.float32)
    if dtype == "bf16":
        a = O.bf16_round(a)
        w = O.bf16_round(w)
        ta = torch.from_numpy(a).to("cuda").to(torch.bfloat16)
        tw = torch.from_numpy(w).to("cuda").to(torch.bfloat16)
        code = binding.ALR_BF16
    else:
        ta, tw = torch.from_numpy(a).cuda(), torch.from_numpy(w).cuda()
        code = binding.ALR_F32
    c = torch.empty((M, N), dtype=torch.float32, device="cuda")
    binding.debug_gemm(code, ta, tw, c, tile=tile)
    torch.cuda.synchronize()
    ref = a.astype(np.float64) @ w.astype(np.float64).T
    err = np.abs(c.cpu().numpy() - ref).max()
    assert err <= 2e-5 * np.sqrt(K) * 4, err


@pytest.mark.parametrize("M", [1, 31, 32, 33, 64, 65, 128, 129, 256])
@pytest.mark.parametrize("N,K", [(64, 64), (192, 192), (320, 1536), (8256, 512)])
def test_gemm_few_rows(M, N, K):
    """The ring kernels at the edges of their row tiles, with fewer K steps than ring stages,
    column tiles that end mid-tile, and more column tiles than CUs, against float64."""
    _print(f"gemm few rows {M}x{N}x{K}")
    rng = np.random.default_rng(M + N + K)
    a = O.bf16_round(rng.standard_normal((M, K)).astype(np.float32))
    w = O.bf16_round(rng.standard_normal((N, K)).astype(np.float32))
    ta, tw = (torch.from_numpy(x).to("cuda").to(torch.bfloat16) for x in (a, w))
    c = torch.empty((M, N), dtype=torch.float32, device="cuda")
    binding.debug_gemm(binding.ALR_BF16, ta, tw, c)
    err = np.abs(c.cpu().numpy() - a.astype(np.float64) @ w.astype(np.float64).T).max()
    assert err <= 2e-5 * np.sqrt(K) * 4, err


@pytest.mark.parametrize("tile", [17, 18, 19, 21])
@pytest.mark.parametrize("M,N,K", [(256, 256, 192), (255, 320, 256), (513, 192, 448),
                                   (4400, 4160, 192), (2560, 7232, 256), (4400, 4160, 704),
                                   (3900, 4352, 1152)])
def test_gemm_wide(M, N, K, tile):
    """The hand-scheduled 256x256 kernel: three and four K steps (the least it takes), odd step
    counts, ragged rows and columns, and more tiles than CUs, so that workgroups go on to a
    second tile whose copies run under the first one's epilogue; on 256 CUs the last two leave 50
    and 16 tiles past the first round, which 21 cuts into 3 and 6 uneven slices; against float64."""
    _print(f"gemm wide tile {tile} {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + K)
    a, w = (torch.randn(s, generator=g).to(torch.bfloat16) for s in ((M, K), (N, K)))
    c = torch.empty((M, N), dtype=torch.float32, device="cuda")
    binding.debug_gemm(binding.ALR_BF16, a.cuda(), w.cuda(), c, tile=tile)
    err = (c.double() - a.cuda().double() @ w.cuda().double().T).abs().max().item()
    assert err <= 2e-5 * np.sqrt(K) * 4, err


@pytest.mark.parametrize("M,N,K", [(7, 64, 64), (8, 128, 512), (9, 192, 320), (1024, 256, 64),
                                   (1025, 256, 64), (4097, 256, 64)])
def test_gemm_f32_few_tiles(M, N, K):
    """fp32 products around the 8-row tiles of the kernel whose waves share K (one wave with work,
    K not a multiple of the waves' share), the last size that takes it (512 tiles) and the first that goes to
    64x64 tiles on 256 CUs, and one with more of those than CUs."""
    _print(f"gemm f32 {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + K)
    a, w = (torch.randn(s, generator=g).cuda() for s in ((M, K), (N, K)))
    c = torch.full((M, N), float("nan"), device="cuda")
    binding.debug_gemm(binding.ALR_F32, a, w, c)
    err = (c.double() - a.double() @ w.double().T).abs().max().item()
    assert err <= 2e-5 * np.sqrt(K) * 4, err


def test_rollout_batches_agree():
    """The first n anchors rolled out alone (ring kernels, each row tile, split and unsplit)
    against the same anchors in a batch of 257 (the tiled kernels), on forced tokens."""
    base = W.get("small_bf16")
    w = W.scaled(base, "batches", n_layers=2, feat_layers=(0, 1), vocab=1024, n_seq=1, seq_len=400,
                 anchors_per_seq=257, anchor_lo=100, anchor_hi=399, block=3)
    inp = W.Inputs(w, W.random_weights(w.shape, 7, scale=0.05, norm_gain="random"),
                   W.random_tokens(1024, (1, 400), 8), *W.random_anchors(1, 400, 257, 100, 399, 9),
                   None, None)
    eng = make_engine(inp)
    prefill(eng, inp)
    forced = torch.from_numpy(W.random_tokens(1024, (257, 3), 10)).cuda()
    _, lp, ft = eng.rollout(inp.anchor_seq, inp.anchor_pos, 3, forced=forced)
    for n in (1, 32, 33, 64, 65, 128, 129, 256):
        _, lpn, ftn = eng.rollout(inp.anchor_seq[:n], inp.anchor_pos[:n], 3, forced=forced[:n])
        # one bf16 rounding of an operand moves by at most 2^-8 of its value
        for x, y in ((lpn, lp[:n]), (ftn, ft[:n])):
            rel = float((x - y).norm() / y.norm())
            assert rel <= 2 ** -8, (n, rel)
        assert torch.equal(ftn[:, 0], ft[:n, 0])  # slot 0 is the prefill's row
    eng.close()


# ------------------------------------------------------------------ fp32 workload
def _full_compare(inp, sel=None, block=None, whole_batch=False):
    """Rolls out the anchors `sel` (whole_batch: every anchor) and compares those of `sel`."""
    w = inp.workload
    block = block or w.block
    n = len(inp.anchor_seq)
    sel = np.arange(n) if sel is None else np.asarray(sel)
    batch = np.arange(n) if whole_batch else sel
    eng = make_engine(inp, max_anchors=len(batch), max_block=block)
    prefill(eng, inp)
    run = runner(eng, inp.anchor_seq[batch], inp.anchor_pos[batch], block)

    def gpu_run(forced):
        if forced is not None and whole_batch:  # the other anchors stay greedy
            every = np.full((n, block), -1, np.int64)
            every[sel] = forced
            forced = every
        out = run(forced)
        return tuple(x[sel] for x in out) if whole_batch else out

    rep = compare(inp, w.shape, sel, gpu_run, block)
    eng.close()
    _print(rep)
    return rep


def test_tiny_fp32_workload_matches_oracle():
    rep = _full_compare(W.make_inputs("tiny_fp32"))
    assert rep.ok()


def test_tiny_fp32_gqa_random_gains():
    base = W.get("tiny_fp32")
    w = W.scaled(base, "tiny_fp32_gqa", n_kv_heads=2, n_heads=4, head_dim=32)
    shape = w.shape
    inp = W.Inputs(w, W.random_weights(shape, 77, norm_gain="random", scale=0.05),
                   W.make_tokens(base), *W.make_anchors(base), None, None)
    rep = _full_compare(inp)
    assert rep.ok()


def test_zero_layer_bf16_iterated_map():
    base = W.get("tiny_fp32")
    w = W.scaled(base, "zero_layer_bf16", n_layers=0, feat_layers=(), dtype="bf16", vocab=1024,
                 d_model=256)
    inp = W.Inputs(w, W.random_weights(w.shape, 5, scale=0.5), W.random_tokens(1024, (1, 128), 3),
                   *W.make_anchors(base), None, None)
    rep = _full_compare(inp)
    assert rep.ok()


@pytest.mark.parametrize("hd,H,G", [(64, 8, 2), (128, 8, 2), (128, 7, 1), (32, 4, 4)])
def test_small_bf16_attention_paths(hd, H, G):
    """Both MFMA attention kernels (hd 64/128, rep 4 and 7) and the generic one (hd 32)."""
    base = W.get("small_bf16")
    w = W.scaled(base, f"small_bf16_{hd}_{H}_{G}", n_layers=2, d_model=256, n_heads=H,
                 n_kv_heads=G, head_dim=hd, d_ffn=512, vocab=2048, feat_layers=(0, 1),
                 n_seq=2, seq_len=300, anchors_per_seq=6, anchor_lo=0, anchor_hi=299, block=5)
    inp = W.Inputs(w, W.random_weights(w.shape, hd + H, scale=0.05, norm_gain="random"),
                   W.random_tokens(2048, (2, 300), 9, dist="zipf"),
                   *W.random_anchors(2, 300, 6, 0, 299, 4), None, None)
    rep = _full_compare(inp)
    assert rep.ok()


@pytest.mark.parametrize("dtype,hd,H,G", [("f32", 96, 4, 2), ("f32", 250, 32, 32), ("bf16", 80, 8, 4),
                                          ("bf16", 36, 32, 16)])
def test_generic_attention_head_sizes(dtype, hd, H, G):
    """The generic attention with 16-byte loads at head sizes that leave lanes of a key idle (96,
    80), with 4- and 8-byte ones where rows do not start on 16 bytes (36 in bf16, 250), rows of
    more keys than one round of its four waves, and a one-key prefix."""
    base = W.get("small_bf16")
    lens = [300, 1]
    w = W.scaled(base, f"generic_{dtype}_{hd}", n_layers=2, d_model=256, n_heads=H, n_kv_heads=G,
                 head_dim=hd, d_ffn=128, vocab=512, feat_layers=(0, 1), dtype=dtype, n_seq=2,
                 seq_len=300, block=4)
    tok = W.random_tokens(512, (2, 300), hd, dist="zipf")
    a_seq, a_pos = np.array([0, 0, 0, 0, 1], np.int32), np.array([0, 63, 254, 299, 0], np.int32)
    inp = W.Inputs(w, W.random_weights(w.shape, hd, scale=0.05, norm_gain="random"), tok, a_seq,
                   a_pos, None, None)
    eng = make_engine(inp, max_anchors=5, max_block=4)
    flat = np.concatenate([tok[s, :n] for s, n in enumerate(lens)]).astype(np.int32)
    eng.prefill(torch.from_numpy(flat).to(eng.device), lens)
    rep = compare(inp, w.shape, np.arange(5), runner(eng, a_seq, a_pos, 4), 4)
    eng.close()
    _print(rep)
    assert rep.ok()


@pytest.mark.parametrize("dtype,hd,H,G,tokens", [("f32", 64, 1, 1, 63), ("f32", 64, 1, 1, 65),
                                                 ("f32", 250, 32, 32, 129), ("f32", 32, 4, 2, 1025),
                                                 ("bf16", 96, 2, 2, 1030), ("bf16", 96, 4, 2, 512)])
def test_generic_attention_waves_per_row(dtype, hd, H, G, tokens):
    """Both forms of the generic attention at the edges of its choice on 256 CUs: a wave per row where no
    row has more than 64 keys (63 items, the last workgroup not full), in bf16 from 2048 items up to 512
    keys (2048, 512), in fp32 from 4096 up to 1024 (4128, head size 250); four waves per row else."""
    base = W.get("small_bf16")
    w = W.scaled(base, f"waves_{dtype}_{hd}_{tokens}", n_layers=2, d_model=256, n_heads=H,
                 n_kv_heads=G, head_dim=hd, d_ffn=128, vocab=512, feat_layers=(0, 1), dtype=dtype,
                 n_seq=1, seq_len=tokens, block=3)
    a_pos = np.array([0, 30, tokens // 2, tokens - 2, tokens - 1], np.int32)
    inp = W.Inputs(w, W.random_weights(w.shape, hd, scale=0.05, norm_gain="random"),
                   W.random_tokens(512, (1, tokens), hd, dist="zipf"), np.zeros(5, np.int32), a_pos,
                   None, None)
    rep = _full_compare(inp)
    assert rep.ok()


def test_generic_attention_past_one_grid_dimension():
    """More (query, head) pairs than one grid dimension holds workgroups of 256 threads (2^24): the
    last sequences repeat the first ones' tokens, so their rows are bit-identical to rows of the first
    2^24 pairs, which the other tests of this kernel cover."""
    base = W.get("tiny_fp32")
    n_seq, length, H = 8080, 65, 32
    w = W.scaled(base, "grid", n_layers=1, d_model=64, n_heads=H, n_kv_heads=H, head_dim=2,
                 d_ffn=64, vocab=64, feat_layers=(0,), n_seq=n_seq, seq_len=length, block=1)
    assert w.n_tokens * H > 1 << 24
    tok = W.random_tokens(64, (n_seq, length), 3)
    tok[-40:] = tok[:40]
    inp = W.Inputs(w, W.random_weights(w.shape, 4, scale=0.3, norm_gain="random"), tok,
                   np.zeros(1, np.int32), np.zeros(1, np.int32), None, None)
    eng = make_engine(inp, max_anchors=1)
    fo = prefill(eng, inp, feats=True).view(n_seq, length, -1)
    torch.cuda.synchronize()
    same = torch.equal(fo[-40:], fo[:40])
    assert same
    eng.close()


def test_generic_attention_tile_of_minus_infinity():
    """A query whose scores against all keys of one wave's tile overflow to -inf (weight 0): keys
    64..127 hold token 1, its key is -1e19 times the query of token 2 along one rotary dim that
    hardly turns; token 0 has a zero key.  The row of token 2 is the mean of the other values."""
    base = W.get("tiny_fp32")
    w = W.scaled(base, "minus_inf", n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, head_dim=64,
                 d_ffn=64, vocab=64, feat_layers=(0,), rope_base=1e9, n_seq=1, seq_len=129, block=1)
    wts = W.random_weights(w.shape, 6, scale=0.3)
    wts["tok_embed"][:] = 0
    for t in range(3):
        wts["tok_embed"][t, t] = 1
    ly = wts["layers"][0]
    for k in ("wq", "wk", "w_down"):
        ly[k][:] = 0
    ly["wk"][31, 1], ly["wq"][31, 2] = -1e19, 1e20
    tok = np.zeros((1, 129), np.int64)
    tok[0, 64:128], tok[0, 128] = 1, 2
    inp = W.Inputs(w, wts, tok, np.zeros(1, np.int32), np.zeros(1, np.int32), None, None)
    eng = make_engine(inp, max_anchors=1)
    row = prefill(eng, inp, feats=True)[128, 0].double().cpu().numpy()
    eng.close()
    f64 = {k: np.asarray(ly[k], np.float64) for k in ("wv", "wo", "attn_norm")}
    e = np.asarray(wts["tok_embed"], np.float64)[:3]
    v = (e / np.sqrt((e * e).mean(1, keepdims=True) + w.shape.rms_eps) * f64["attn_norm"]) @ f64["wv"].T
    want = e[2] + f64["wo"] @ ((64 * v[0] + v[2]) / 65)
    # 65 equal weights and 64 products per output, in 32 bits
    np.testing.assert_allclose(row, want, rtol=0, atol=1e-5 * np.abs(want).max())


@pytest.mark.parametrize("hd,H,G,tokens,kernel", [(36, 32, 16, 90, 6), (100, 16, 16, 90, 6),
                                                  (10, 64, 32, 90, 6), (50, 32, 32, 64, 1),
                                                  (50, 32, 32, 200, 4), (50, 32, 32, 1000, 5)])
def test_rope_pairs_across_heads(hd, H, G, tokens, kernel):
    """bf16 head sizes whose half is no multiple of 4 (36, 100) or odd (50, 10): runs of four and
    pairs of neighbouring columns of the fused QKV product then cross from one head into the next,
    in the split-K reduce of the rollout and in the row epilogues of the prefill (the few-row
    kernel, the LDS-staged one of both tiles, 256x256 tiles)."""
    base = W.get("small_bf16")
    w = W.scaled(base, f"pairs_{hd}_{tokens}", n_layers=2, d_model=2048, n_heads=H, n_kv_heads=G,
                 head_dim=hd, d_ffn=128, vocab=512, feat_layers=(0, 1), n_seq=2,
                 seq_len=tokens, block=4)
    lim = binding.make_limits(w.n_tokens, 2, 5, 4)
    _, splits, _ = binding.gemm_plan(w.shape, lim, "decode_qkv", 5, n_cu=n_cu())
    assert splits > 1
    assert binding.gemm_plan(w.shape, lim, "prefill_qkv", w.n_tokens, n_cu=n_cu())[0] == kernel
    a_seq = np.array([0, 0, 1, 1, 1], np.int32)
    a_pos = np.array([0, 40, 33, tokens // 2, tokens - 1], np.int32)
    inp = W.Inputs(w, W.random_weights(w.shape, hd, scale=0.02, norm_gain="random"),
                   W.random_tokens(512, (2, tokens), hd, dist="zipf"), a_seq, a_pos, None, None)
    rep = _full_compare(inp)
    assert rep.ok()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_wide_residual_rows(dtype):
    """d_model 8448: rows wider than the 8192 elements RMSNorm holds in registers, so every norm
    also runs its streaming tail; the GEMMs see K = 8448 and 33 column tiles of 256, and in bf16
    the rollout's down projection (66 rows, K = 1024) is split over K with rows too wide for the
    reduce fused with the next norm, so the plain reduce and a separate norm run."""
    base = W.get("small_bf16")
    w = W.scaled(base, f"wide_{dtype}", n_layers=1, d_model=8448, n_heads=4, n_kv_heads=1,
                 head_dim=64, d_ffn=1024, vocab=512, feat_layers=(0,), dtype=dtype, n_seq=2,
                 seq_len=96, anchors_per_seq=33, anchor_lo=0, anchor_hi=95, block=4)
    if dtype == "bf16":
        _, splits, _ = binding.gemm_plan(w.shape, binding.make_limits(192, 2, 66, 4),
                                         "decode_down", 66, n_cu=n_cu())
        assert splits == 2
    inp = W.Inputs(w, W.random_weights(w.shape, 8448, scale=0.02, norm_gain="random"),
                   W.random_tokens(512, (2, 96), 29, dist="zipf"),
                   *W.random_anchors(2, 96, 33, 0, 95, 12), None, None)
    rep = _full_compare(inp, sel=np.array([0, 16, 32, 33, 50, 65]), whole_batch=True)
    assert rep.ok()


def test_small_bf16_workload_subset():
    inp = W.make_inputs("small_bf16")
    sel = np.array([0, 1, 70, 130, 200, 255])
    rep = _full_compare(inp, sel=sel)
    assert rep.ok()


@pytest.mark.parametrize("dtype,hd,H,G", [("bf16", 128, 8, 2), ("bf16", 64, 8, 2), ("f32", 32, 4, 2)])
def test_ragged_sequences_and_edge_anchors(dtype, hd, H, G):
    """One prefill over sequences of ragged lengths (300, 129, 64 and 1 tokens: partial key tiles,
    a one-token prefix); anchors at each sequence's first and last position, one anchor twice, and
    rollout positions past the sequence end."""
    lens = [300, 129, 64, 1]
    base = W.get("small_bf16")
    w = W.scaled(base, f"ragged_{dtype}_{hd}", n_layers=2, d_model=256, n_heads=H, n_kv_heads=G,
                 head_dim=hd, d_ffn=512, vocab=2048, feat_layers=(0, 1), dtype=dtype,
                 n_seq=len(lens), seq_len=max(lens), block=5)
    tok_pad = W.random_tokens(2048, (len(lens), max(lens)), 17 + hd, dist="zipf")
    a_seq = np.array([0, 0, 0, 1, 1, 1, 2, 2, 3, 1], np.int32)
    a_pos = np.array([0, 299, 150, 0, 128, 128, 63, 31, 0, 64], np.int32)
    inp = W.Inputs(w, W.random_weights(w.shape, 31 + hd, scale=0.05, norm_gain="random"),
                   tok_pad, a_seq, a_pos, None, None)
    eng = make_engine(inp, max_anchors=len(a_seq), max_block=w.block)
    flat = np.concatenate([tok_pad[s, :n] for s, n in enumerate(lens)]).astype(np.int32)
    eng.prefill(torch.from_numpy(flat).to(eng.device), lens)
    rep = compare(inp, w.shape, np.arange(len(a_seq)), runner(eng, a_seq, a_pos, w.block), w.block)
    eng.close()
    _print(rep)
    assert rep.ok()


# ------------------------------------------------------------------ invariants (bit-exact)
def test_permutation_duplicates_and_slot0():
    inp = W.make_inputs("tiny_fp32")
    w = inp.workload
    eng = make_engine(inp, max_anchors=3 * w.n_anchors)
    fo = prefill(eng, inp, feats=True)
    a_s, a_p = inp.anchor_seq, inp.anchor_pos
    run = runner(eng, a_s, a_p, w.block)
    t0, l0, f0 = run(None)
    perm = np.random.default_rng(1).permutation(w.n_anchors)
    t1, l1, f1 = runner(eng, a_s[perm], a_p[perm], w.block)(None)
    np.testing.assert_array_equal(t1, t0[perm])
    np.testing.assert_array_equal(l1, l0[perm])
    np.testing.assert_array_equal(f1, f0[perm])
    dup = np.concatenate([np.arange(w.n_anchors), np.arange(w.n_anchors)[::-1]])
    t2, l2, f2 = runner(eng, a_s[dup], a_p[dup], w.block)(None)
    np.testing.assert_array_equal(t2, t0[dup])
    np.testing.assert_array_equal(l2, l0[dup])
    # slot-0 features equal the prefill's features at the anchor
    fpre = fo.cpu().numpy()
    np.testing.assert_array_equal(f0[:, 0], fpre[w.seq_len * a_s + a_p])
    eng.close()


def test_forced_corpus_continuation_matches_later_anchor_slot0():
    """Feeding the corpus continuation makes slot s of anchor a the prefill output at a+s."""
    inp = W.make_inputs("tiny_fp32")
    w = inp.workload
    a_p = np.array([10, 40, 77], np.int32)
    a_s = np.zeros(3, np.int32)
    B = 4
    eng = make_engine(inp, max_anchors=16, max_block=B)
    prefill(eng, inp)
    forced = np.stack([inp.tokens[0, a + 1:a + 1 + B] for a in a_p]).astype(np.int32)
    t, lp, ft = runner(eng, a_s, a_p, B)(forced)
    later_p = np.array([a + s for a in a_p for s in range(B)], np.int32)
    t0, lp0, ft0 = runner(eng, np.zeros(len(later_p), np.int32), later_p, 1)(None)
    np.testing.assert_allclose(lp.reshape(-1, w.shape.vocab), lp0[:, 0], atol=2e-5, rtol=0)
    np.testing.assert_allclose(ft.reshape(len(later_p), w.shape.n_feat, -1), ft0[:, 0], atol=2e-5,
                               rtol=0)
    eng.close()


@pytest.mark.parametrize("dtype,hd", [("bf16", 128), ("f32", 32)])
def test_second_prefill_replaces_the_first(dtype, hd):
    """A context reused for a second corpus (other lengths and tokens, after a rollout of the first)
    gives bit-identical rollouts to a fresh context: nothing of the first prefill, its cache layout
    or its rollout plan leaks into the second."""
    base = W.get("small_bf16")
    w = W.scaled(base, f"reuse_{dtype}_{hd}", n_layers=2, d_model=256, n_heads=8, n_kv_heads=2,
                 head_dim=hd, d_ffn=512, vocab=2048, feat_layers=(0, 1), dtype=dtype, n_seq=3,
                 seq_len=300, block=5)
    wts = W.random_weights(w.shape, 7 + hd, scale=0.05, norm_gain="random")
    lens_a, lens_b = [300, 200, 100], [129, 300]
    tok_a = W.random_tokens(2048, (3, 300), 1, dist="zipf")
    tok_b = W.random_tokens(2048, (2, 300), 2, dist="zipf")
    a_s_a, a_p_a = np.array([0, 1, 2, 0], np.int32), np.array([299, 150, 50, 10], np.int32)
    a_s_b, a_p_b = np.array([1, 0, 1, 0], np.int32), np.array([299, 128, 0, 64], np.int32)
    inp = W.Inputs(w, wts, tok_a, a_s_a, a_p_a, None, None)

    def pf(e, tok, lens):
        flat = np.concatenate([tok[q, :n] for q, n in enumerate(lens)]).astype(np.int32)
        e.prefill(torch.from_numpy(flat).to(e.device), lens)

    eng = make_engine(inp, max_anchors=8, max_block=w.block)
    pf(eng, tok_a, lens_a)
    runner(eng, a_s_a, a_p_a, w.block)(None)
    pf(eng, tok_b, lens_b)
    t1, l1, f1 = runner(eng, a_s_b, a_p_b, w.block)(None)
    eng.close()
    fresh = make_engine(inp, max_anchors=8, max_block=w.block)
    pf(fresh, tok_b, lens_b)
    t2, l2, f2 = runner(fresh, a_s_b, a_p_b, w.block)(None)
    fresh.close()
    np.testing.assert_array_equal(t1, t2)
    np.testing.assert_array_equal(l1, l2)
    np.testing.assert_array_equal(f1, f2)


def test_rollout_before_prefill_is_a_state_error():
    inp = W.make_inputs("tiny_fp32")
    eng = make_engine(inp)
    with pytest.raises(binding.AlrError) as e:
        eng.rollout(inp.anchor_seq, inp.anchor_pos, 4)
    assert e.value.status == 4
    eng.close()
