"""GPU parity: causal prefill attention vs the oracle's exact softmax(QK^T)V."""
import numpy as np
import pytest
import torch

import vitcop_inputs as I
from oracle import vitcop_oracle as O
from gpu_util import assert_attention_close, dev, host_bits, host_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vc():
    from paper_2601_17818_amd import binding
    return binding


def run(vc, t, causal=True, scale=0.0, lse=True):
    out, l = vc.vitcop_prefill_attn(dev(t["q"]), dev(t["k"]), dev(t["v"]), scale, causal, lse)
    torch.cuda.synchronize()
    return host_f64(out), (l.cpu().numpy().astype(np.float64) if lse else None)


# N spans: single row, inside one 32-row wavefront tile, exactly one key tile, ragged
# tails, several query blocks
@pytest.mark.parametrize("N", [1, 2, 31, 32, 33, 64, 65, 100, 127, 128, 129, 191, 300, 517])
def test_causal_sizes(vc, N):
    t = I.qkv_tensors(100 + N, 2, N, 3, 3, 128)
    out, lse = run(vc, t)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"])
    assert_attention_close(out, ref, f"N={N}")
    assert np.abs(lse - ref_lse).max() < 1e-3


# with few heads a wavefront owns one 32-query block at every length: block edges (128 queries per workgroup),
# ragged tails, several blocks, more key tiles than the ring has stages
@pytest.mark.parametrize("N", [320, 321, 384, 500, 511, 512, 513, 640, 784, 1024, 1025, 1087, 1280, 1500, 2100])
def test_causal_long(vc, N):
    t = I.qkv_tensors(150 + N, 1, N, 2, 2, 128)
    out, lse = run(vc, t)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"])
    assert_attention_close(out, ref, f"N={N}")
    assert np.abs(lse - ref_lse).max() < 1e-3


# enough (sample, head) pairs that 256-query workgroups fill the chip: from 512 tokens on a wavefront then owns
# two 32-query blocks.  Block edges, ragged first blocks, GQA, and the case just below the switch (one block)
@pytest.mark.parametrize("B,N,Hq,Hkv,causal", [
    (5, 512, 28, 4, True), (5, 513, 28, 4, True), (3, 777, 24, 24, True), (2, 1025, 28, 4, True),
    (2, 1300, 24, 8, True), (2, 1300, 24, 8, False), (5, 511, 28, 4, True), (1, 1025, 28, 4, True)])
def test_many_heads_two_query_blocks_per_wavefront(vc, B, N, Hq, Hkv, causal):
    t = I.qkv_tensors(170 + N + B, B, N, Hq, Hkv, 128)
    out, lse = run(vc, t, causal=causal)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], None, causal)
    assert_attention_close(out, ref, f"B={B} N={N} {Hq}/{Hkv} causal={causal}")
    assert np.abs(lse - ref_lse).max() < 1e-3


def test_long_gqa_batch_and_non_causal(vc):
    t = I.qkv_tensors(160, 2, 1111, 8, 2, 128)
    out, lse = run(vc, t)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"])
    assert_attention_close(out, ref, "long GQA")
    assert np.abs(lse - ref_lse).max() < 1e-3
    t = I.qkv_tensors(161, 1, 1300, 2, 1, 128)
    out, lse = run(vc, t, causal=False)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], None, False)
    assert_attention_close(out, ref, "long non-causal")
    assert np.abs(lse - ref_lse).max() < 1e-3


def test_long_large_logits(vc):
    # logits of order +-100 with outliers: exercises the deferred rescaling of the accumulators
    t = I.qkv_tensors(162, 1, 1200, 2, 2, 128, std=3.0)
    out, lse = run(vc, t, scale=0.11)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], 0.11)
    assert_attention_close(out, ref, "long large logits", v_scale=3.0)
    assert np.abs(lse - ref_lse).max() < 2e-3 * max(1.0, np.abs(ref_lse).max())


@pytest.mark.parametrize("N,d,H", [(1500, 128, 2), (300, 128, 2), (700, 64, 2), (1040, 128, 56)])
def test_rising_scores_move_the_reference(vc, N, d, H):
    # scores that climb along the keys by several hundred in the exponent: the kernels raise their reference
    # maximum again and again (and rescale what they have accumulated), also inside diagonal tiles; softmax
    # weight sits on the last visible keys, so every row checks the state after all those moves
    # (56 heads: two query blocks per wavefront, each with a reference of its own)
    g = np.random.default_rng(77 + N)
    q = np.ones((1, N, H, d), np.float32) + 0.05 * g.standard_normal((1, N, H, d)).astype(np.float32)
    ramp = (np.arange(N, dtype=np.float32) / N * 6.0)[None, :, None, None]
    k = ramp * np.ones((1, N, H, d), np.float32) + 0.05 * g.standard_normal((1, N, H, d)).astype(np.float32)
    t = {"q": I.f32_to_bf16_bits(q), "k": I.f32_to_bf16_bits(k), "v": I.normal_bf16(78 + N, 3, (1, N, H, d))}
    out, lse = run(vc, t)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"])
    assert ref_lse.max() - ref_lse.min() > 40.0                  # the logits do span hundreds of bits
    assert_attention_close(out, ref, f"rising scores N={N} d={d}")
    assert np.abs(lse - ref_lse).max() < 2e-3 * max(1.0, np.abs(ref_lse).max())


@pytest.mark.parametrize("N", [5, 64, 130, 257])
def test_non_causal(vc, N):
    t = I.qkv_tensors(200 + N, 1, N, 2, 2, 128)
    out, lse = run(vc, t, causal=False)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], None, False)
    assert_attention_close(out, ref, f"non-causal N={N}")
    assert np.abs(lse - ref_lse).max() < 1e-3


# one to eight keys past the last whole tile of 64 go without a tile (9 and none beside them), d = 64
@pytest.mark.parametrize("N", [64, 65, 66, 68, 69, 72, 73, 129, 197, 260, 577, 584, 585])
@pytest.mark.parametrize("std", [1.0, 3.0])
def test_keys_past_the_last_tile(vc, N, std):
    t = I.qkv_tensors(210 + N, 2, N, 4, 2, 64, std=std)
    for last in (1.0, 4.0):          # (the last keys' scores like the others', and far above or below them)
        k = I.bf16_bits_to_f32(t["k"])
        k[:, N - N % 64:] *= last
        t["k"] = I.f32_to_bf16_bits(k)
        out, lse = run(vc, t, causal=False)
        ref, ref_lse = O.attention(t["q"], t["k"], t["v"], None, False)
        assert_attention_close(out, ref, f"N={N}", v_scale=std)
        assert np.abs(lse - ref_lse).max() < 1e-3 * max(1.0, np.abs(ref_lse).max() / 10)


# One key of the tiles holds nearly all of the weight, a key past them lies five binary orders below.  The large probability
# is exact if it is the reference (its weight rounded to bf16 is off by up to 2^-9, which moves every second output); what
# is left are the other keys' roundings, 2^-9 of a twentieth of the weight, which move one output in twenty or so.
@pytest.mark.parametrize("N", [65, 72, 129, 260])
def test_the_largest_weight_is_exact_beside_keys_past_the_last_tile(vc, N):
    g = torch.Generator(device="cuda").manual_seed(N)
    e = torch.empty(64, device="cuda").normal_(generator=g)
    e = e / e.norm()
    unit = 8.0 / 1.4426950408889634                          # a score of one in powers of two
    k = torch.empty((2, N, 4, 64), device="cuda").normal_(0, 0.1, generator=g)
    k[:, 20] = 13.0 * unit * e
    k[:, N - 1] = 8.0 * unit * e
    q = e * torch.empty((2, N, 4, 1), device="cuda").uniform_(0.9, 1.1, generator=g)
    v = torch.empty((2, N, 4, 64), device="cuda").normal_(generator=g)
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    out = vc.vitcop_prefill_attn(q, k, v, causal=False)[0]
    qd, kd, vd = (t.double().cpu().permute(0, 2, 1, 3).contiguous() for t in (q, k, v))
    p = torch.softmax(qd @ kd.transpose(2, 3).contiguous() / 8.0, dim=-1)
    assert float(p[..., 20].min()) > 0.85
    want = (p @ vd).permute(0, 2, 1, 3).float().bfloat16()
    assert float((out.cpu() == want).float().mean()) > 0.85


# a NaN in the last key reaches every query of its heads, whether that key stands alone past the last tile or not
@pytest.mark.parametrize("N", [64, 65, 66, 72, 73])
def test_nan_in_the_last_key(vc, N):
    t = I.qkv_tensors(240 + N, 1, N, 4, 2, 64)
    t["k"][0, N - 1, 1] = 0x7FC0
    out, _ = run(vc, t, causal=False)
    assert np.isnan(out[0, :, 2:]).all() and np.isfinite(out[0, :, :2]).all()


# the same for any key, both head dimensions, one and two query blocks to a wavefront (two: 1100 tokens of 128 channels) and
# with the mask, where the queries before that key do not see it
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,at", [(64, 0), (65, 64), (300, 0), (300, 31), (300, 32), (577, 576), (577, 575), (700, 130), (1100, 1099)])
def test_nan_in_a_key_reaches_the_queries_that_see_it(vc, causal, d, N, at):
    B, Hq = (1, 4) if N < 1000 else (4, 32)
    g = torch.Generator(device="cuda").manual_seed(N + at)
    q, k, v = (torch.empty((B, N, h, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for h in (Hq, Hq // 2, Hq // 2))
    want = vc.vitcop_prefill_attn(q, k, v, causal=causal)[0].clone()
    k[0, at, 1, 3] = float("nan")
    out = vc.vitcop_prefill_attn(q, k, v, causal=causal)[0]
    first = at if causal else 0
    assert bool(out[0, first:, 2:4].isnan().all())
    out[0, first:, 2:4] = want[0, first:, 2:4]
    assert torch.equal(out, want)


@pytest.mark.parametrize("Hq,Hkv", [(28, 4), (8, 2), (6, 1)])
def test_gqa(vc, Hq, Hkv):
    t = I.qkv_tensors(300 + Hq, 1, 150, Hq, Hkv, 128)
    out, _ = run(vc, t)
    ref, _ = O.attention(t["q"], t["k"], t["v"])
    assert_attention_close(out, ref, f"GQA {Hq}/{Hkv}")


def test_explicit_scale_and_large_logits(vc):
    t = I.qkv_tensors(400, 1, 140, 2, 2, 128, std=3.0)       # logits of order +-100
    out, lse = run(vc, t, scale=0.11)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], 0.11)
    assert_attention_close(out, ref, "large logits", v_scale=3.0)
    assert np.abs(lse - ref_lse).max() < 2e-3 * max(1.0, np.abs(ref_lse).max())


def test_structure_pins(vc):
    t = I.qkv_tensors(500, 1, 200, 2, 2, 128)
    ones = I.f32_to_bf16_bits(np.ones((1, 200, 2, 128), np.float32))
    out, _ = run(vc, dict(t, v=ones))
    assert np.abs(out - 1.0).max() < 1e-2                       # rows of softmax sum to 1
    out, _ = run(vc, t)
    v = I.bf16_bits_to_f32(t["v"]).astype(np.float64)
    assert np.array_equal(out[0, 0], v[0, 0])                   # row 0 sees key 0 only
    kk = np.tile(t["k"][:, :1], (1, 200, 1, 1))
    out, _ = run(vc, dict(t, k=kk))
    run_mean = np.cumsum(v[0], axis=0) / np.arange(1, 201)[:, None, None]
    assert np.abs(out[0] - run_mean).max() < 2e-2


def test_config0_pruned_shape_and_unpruned_shape(vc):
    for N in (128, 640):
        t = I.qkv_tensors(600 + N, 1, N, 32, 32, 128)
        out, lse = run(vc, t)
        ref, ref_lse = O.attention(t["q"], t["k"], t["v"])
        assert_attention_close(out, ref, f"config0 N={N}")
        assert np.abs(lse - ref_lse).max() < 1e-3


# head dimension 64 (the vision encoder's, and small language models')
@pytest.mark.parametrize("N", [1, 33, 64, 65, 129, 300, 577, 1111])
def test_head_dim_64_causal(vc, N):
    t = I.qkv_tensors(800 + N, 2, N, 4, 2, 64)
    out, lse = run(vc, t)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"])
    assert_attention_close(out, ref, f"d=64 N={N}")
    assert np.abs(lse - ref_lse).max() < 1e-3


def test_head_dim_64_non_causal_and_scale(vc):
    t = I.qkv_tensors(850, 1, 577, 16, 16, 64)                  # one CLIP-L image: 576 patches + [CLS]
    out, lse = run(vc, t, causal=False)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], None, False)
    assert_attention_close(out, ref, "d=64 non-causal")
    assert np.abs(lse - ref_lse).max() < 1e-3
    t = I.qkv_tensors(851, 1, 200, 2, 2, 64, std=3.0)
    out, lse = run(vc, t, scale=0.2)
    ref, ref_lse = O.attention(t["q"], t["k"], t["v"], 0.2)
    assert_attention_close(out, ref, "d=64 large logits", v_scale=3.0)
    assert np.abs(lse - ref_lse).max() < 2e-3 * max(1.0, np.abs(ref_lse).max())


def test_deterministic(vc):
    t = I.qkv_tensors(700, 2, 300, 4, 2, 128)
    q, k, v = dev(t["q"]), dev(t["k"]), dev(t["v"])
    a, _ = vc.vitcop_prefill_attn(q, k, v)
    for _ in range(5):
        b, _ = vc.vitcop_prefill_attn(q, k, v)
        assert torch.equal(a, b)


# what the pipelined kernel cannot address goes to the kernel with a three-dimensional grid and 64-bit offsets
def test_more_workgroups_than_one_grid_dimension_holds(vc):
    B, Hq = 65535, 260                                   # 17 million (sample, head) pairs of one token each
    q = torch.ones((B, 1, Hq, 64), dtype=torch.bfloat16, device="cuda")
    k, v = (torch.empty((B, 1, 1, 64), dtype=torch.bfloat16, device="cuda").normal_() for _ in range(2))
    out, _ = vc.vitcop_prefill_attn(q, k, v)
    assert bool((out == v).all())                        # a softmax over one key


@pytest.mark.parametrize("d,H,N,causal", [(64, 31552, 1000, True), (64, 33600, 960, False), (128, 15776, 1000, True)])
def test_keys_beyond_32_bit_offsets(vc, d, H, N, causal):
    assert (N + 64) * H * d * 2 >= 1 << 32
    g = torch.Generator(device="cuda").manual_seed(d + N)
    q, k, v = (torch.empty((1, N, H, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(3))
    out, lse = vc.vitcop_prefill_attn(q, k, v, causal=causal, want_lse=True)
    heads = [0, 1, H // 2, H - 1]
    t = [host_bits(x[:, :, heads]) for x in (q, k, v)]
    ref, ref_lse = O.attention(*t, None, causal)
    assert_attention_close(host_f64(out[:, :, heads]), ref, f"d={d} N={N}")
    assert np.abs(lse[:, heads].cpu().numpy() - ref_lse).max() < 1e-3
