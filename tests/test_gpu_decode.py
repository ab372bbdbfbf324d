"""GPU parity: one decoding step over a (compacted) KV cache vs the oracle's softmax(K q) V."""
import numpy as np
import pytest
import torch

import vitcop_inputs as I
from oracle import decoder_oracle as Dc
from gpu_util import assert_attention_close, dev, host_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vc():
    from paper_2601_17818_amd import binding
    return binding


def run(vc, t, scale=0.0):
    q = dev(t["q"][:, -1])
    o, lse = vc.vitcop_decode_attn(q, dev(t["k"]), dev(t["v"]), scale)
    torch.cuda.synchronize()
    return host_f64(o), lse.cpu().numpy().astype(np.float64)


# cache lengths: one key, inside one lane group, slice edges (64), ragged, several slices;
# head layouts: MHA, the video model's 28/4, a group above 8, d = 64
@pytest.mark.parametrize("B,N,Hq,Hkv,d", [(1, 1, 2, 2, 128), (2, 3, 4, 2, 128), (2, 64, 4, 4, 128), (1, 65, 6, 2, 64),
                                          (3, 384, 32, 32, 128), (1, 755, 28, 4, 128), (2, 1000, 20, 2, 128),
                                          (1, 2944, 8, 8, 128), (4, 224, 16, 16, 64), (1, 6400, 28, 4, 128)])
def test_matches_oracle(vc, B, N, Hq, Hkv, d):
    t = I.qkv_tensors(9500 + N + Hq, B, N, Hq, Hkv, d)
    out, lse = run(vc, t)
    ref, ref_lse = Dc.decode_attention(t["q"][:, -1], t["k"], t["v"])
    assert_attention_close(out, ref, f"decode N={N}")
    assert np.abs(lse - ref_lse).max() < 1e-3


# enough workgroups that two or four heads are read side by side, or one (27 heads, 1040 and 1280 pairs): one key, fewer
# than a round of the wavefronts, a round and one over, several slices with a short last one, rows requested ahead and not
@pytest.mark.parametrize("B,N,H,d", [(32, 1, 32, 128), (32, 33, 32, 128), (8, 200, 32, 128), (32, 65, 32, 64), (32, 1030, 32, 64),
                                     (64, 1, 32, 128), (64, 17, 32, 128), (128, 65, 16, 128), (64, 33, 32, 64),
                                     (64, 1030, 32, 64), (64, 50, 27, 128), (26, 20, 40, 128), (40, 20, 32, 64)])
def test_heads_side_by_side(vc, B, N, H, d):
    # three different samples dealt out at random, and every sample's result against its own
    t = I.qkv_tensors(9900 + N + H, 3, N, H, H, d)
    of = np.random.default_rng(B + N).integers(0, 3, B)
    out, lse = run(vc, {n: x[of] for n, x in t.items()})
    ref, ref_lse = Dc.decode_attention(t["q"][:, -1], t["k"], t["v"])
    assert_attention_close(out, ref[of], f"decode N={N}")
    assert np.abs(lse - ref_lse[of]).max() < 1e-3


# query heads that share a KV head: 2, 3, 7, 16 and 17 of them (a second pass), tiles of 32 keys a wavefront and 128 a
# workgroup short of full, full and one over, one slice and several
@pytest.mark.parametrize("B,N,Hq,Hkv,d", [(2, 31, 4, 2, 64), (2, 32, 6, 2, 128), (1, 33, 7, 1, 64), (3, 127, 16, 1, 128),
                                          (2, 129, 17, 1, 64), (70, 160, 28, 4, 128), (1, 257, 34, 2, 128)])
def test_grouped_query_heads(vc, B, N, Hq, Hkv, d):
    t = I.qkv_tensors(9700 + N + Hq, B, N, Hq, Hkv, d)
    out, lse = run(vc, t)
    ref, ref_lse = Dc.decode_attention(t["q"][:, -1], t["k"], t["v"])
    assert_attention_close(out, ref, f"decode N={N}, {Hq} / {Hkv}")
    assert np.abs(lse - ref_lse).max() < 1e-3


def test_grouped_query_heads_with_infinities(vc):
    # an infinite value reaches its channel of every head and no other; keys whose scores are -inf count for nothing
    B, N, Hq, Hkv, d = 1, 200, 8, 2, 128
    t = I.qkv_tensors(9800, B, N, Hq, Hkv, d)
    plain, _ = run(vc, t)
    v = t["v"].copy()
    v[0, 77, 1, 5] = 0x7F80                                       # +inf in the second KV head's channel 5
    out, _ = run(vc, dict(t, v=v))
    want = plain.reshape(B, Hkv, Hq // Hkv, d).copy()
    want[0, 1, :, 5] = np.inf
    assert np.array_equal(out.reshape(want.shape), want)
    q, k = t["q"].copy(), t["k"].copy()
    q[:, -1, :, 0] = 0x3F80                                       # 1.0
    k[0, :64, :, 0] = 0xFF80                                      # -inf: the first 64 keys, two whole tiles
    out, lse = run(vc, dict(t, q=q, k=k))
    rest = dict(t, q=q, k=k[:, 64:], v=t["v"][:, 64:])
    ref, ref_lse = run(vc, {n: np.ascontiguousarray(x) for n, x in rest.items()})
    assert np.abs(out - ref).max() < 1e-2 and np.abs(lse - ref_lse).max() < 1e-3


# two query heads to a KV head, on both sides of each line between the vector and the matrix-core kernel: few pairs (16 keys),
# up to 64 keys by their number, many pairs (of 64 channels: from 129 keys on and up to 16)
@pytest.mark.parametrize("B,N,Hkv,d", [(2, 1, 2, 128), (2, 16, 2, 128), (2, 17, 2, 128), (34, 34, 16, 128), (33, 34, 16, 128),
                                       (64, 64, 16, 128), (64, 65, 16, 128), (193, 65, 16, 128), (192, 66, 16, 128),
                                       (193, 16, 16, 64), (193, 17, 16, 64), (193, 129, 16, 64), (192, 129, 16, 64)])
def test_two_query_heads_to_a_kv_head(vc, B, N, Hkv, d):
    t = I.qkv_tensors(9750 + N + B, B, N, 2 * Hkv, Hkv, d)
    out, lse = run(vc, t)
    ref, ref_lse = Dc.decode_attention(t["q"][:, -1], t["k"], t["v"])
    assert_attention_close(out, ref, f"decode N={N}, {2 * Hkv} / {Hkv}")
    assert np.abs(lse - ref_lse).max() < 1e-3


# the newest row of a cache is the last of its slice's last, partly filled tile (of 32 keys a wavefront; with one query head
# per KV head: of the keys of a load, where heads are read one, two and four at a time, slices long and short)
@pytest.mark.parametrize("B,N,Hq,Hkv,d", [(1, 1, 8, 2, 128), (1, 31, 8, 2, 64), (2, 129, 8, 2, 128), (1, 200, 8, 2, 128),
                                          (1, 257, 14, 2, 64), (40, 165, 28, 4, 128), (1, 129, 34, 2, 128),
                                          (1, 201, 2, 2, 128), (1, 203, 4, 4, 64), (32, 33, 32, 32, 128),
                                          (64, 33, 32, 32, 128), (32, 37, 32, 32, 64), (128, 67, 16, 16, 64),
                                          (32, 1029, 32, 32, 64), (2, 15, 4, 2, 128), (64, 31, 16, 8, 128),
                                          (193, 131, 32, 16, 64)])
def test_an_infinite_value_in_the_last_row(vc, B, N, Hq, Hkv, d):
    # it reaches its channel of every head of its KV head, and nothing else: the slots past the last key count for nothing
    t = I.qkv_tensors(9850 + N + Hq, 1, N, Hq, Hkv, d)
    t = {n: np.repeat(x, B, axis=0) for n, x in t.items()}
    plain, plain_lse = run(vc, t)
    v = t["v"].copy()
    v[B - 1, N - 1, Hkv - 1, 5] = 0x7F80                          # +inf
    out, lse = run(vc, dict(t, v=v))
    want = plain.reshape(B, Hkv, Hq // Hkv, d).copy()
    want[B - 1, Hkv - 1, :, 5] = np.inf
    assert np.array_equal(out.reshape(want.shape), want)
    assert np.array_equal(lse, plain_lse)


def test_scale_large_logits_and_structure(vc):
    t = I.qkv_tensors(9600, 2, 300, 4, 2, 128, std=3.0)
    out, lse = run(vc, t, scale=0.11)
    ref, ref_lse = Dc.decode_attention(t["q"][:, -1], t["k"], t["v"], 0.11)
    assert_attention_close(out, ref, "decode large logits", v_scale=3.0)
    assert np.abs(lse - ref_lse).max() < 2e-3 * max(1.0, np.abs(ref_lse).max())
    ones = I.f32_to_bf16_bits(np.ones((2, 300, 2, 128), np.float32))
    out, _ = run(vc, dict(t, v=ones))
    assert np.abs(out - 1.0).max() < 1e-2                         # softmax weights sum to 1


def test_decode_equals_last_row_of_prefill_and_is_deterministic(vc):
    t = I.qkv_tensors(9700, 2, 500, 8, 2, 128)
    q, k, v = dev(t["q"]), dev(t["k"]), dev(t["v"])
    full, _ = vc.vitcop_prefill_attn(q, k, v)
    o, _ = vc.vitcop_decode_attn(q[:, -1].contiguous(), k, v)
    torch.cuda.synchronize()
    assert (full[:, -1].float() - o.float()).abs().max().item() <= 2e-2
    for _ in range(3):
        o2, _ = vc.vitcop_decode_attn(q[:, -1].contiguous(), k, v)
        assert torch.equal(o, o2)
