"""Decode attention at the ends of the fp32 range (Sec. II-B, Eq. (1): a block's exponent byte spans all
of fp32; Sec. III: attention reads the blocks as they are).  The matrix-core passes rescale by powers of
two internally; cached magnitudes from 2^-120 to 2^110 and the matching softmax scales must come out
within the ordinary bar against the oracle, for every kernel family (LDS pipeline, register-staged
4-bit, 8-bit, fp32 I/O)."""
import numpy as np
import pytest
import torch

from oracle import kvbfp_oracle as O
from paper_2403_20137_amd import kvbfp, synth
from util import DT_NAME, assert_attention_close, assert_planes_equal, gpu_cache, oracle_cache

pytestmark = pytest.mark.gpu
D = 128

FAMILIES = [(torch.bfloat16, 32, 4), (torch.bfloat16, 16, 4), (torch.float16, 32, 4), (torch.bfloat16, 128, 4),
            (torch.bfloat16, 16, 8), (torch.float32, 32, 4), (torch.float32, 64, 8)]


def _run(dtype, n, p, k_shift, v_shift, q_shift, compensate=True, G=4):
    """K, V, q drawn as usual, multiplied by 2^shift (exact), rounded to dtype; with `compensate` the softmax
    scale takes the inverse of the key and query shifts, so the logits stay where they were."""
    B, S, Hkv, S_max = 2, 600, 2, 1100
    g = synth.outlier_gains(5, 0, Hkv, D)
    mk = lambda t, sh: (t * 2.0 ** sh).to(dtype)
    k = mk(synth.kv_rows(B, S, Hkv, D, "f32", g, 5, 2), k_shift)
    v = mk(synth.kv_rows(B, S, Hkv, D, "f32", g, 5, 3), v_shift)
    q = mk(synth.queries(B, Hkv * G, D, "f32", 5, 4), q_shift)
    assert bool(torch.isfinite(k).all() and torch.isfinite(v).all() and torch.isfinite(q).all())
    planes = oracle_cache(k, v, n, p, S_max, 0)
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S_max)
    assert_planes_equal(cache, planes, "cache at the end of the range")
    scale = float(np.float32(D ** -0.5) * np.float32(2.0 ** (-(k_shift + q_shift) if compensate else 0)))
    lens = [S, 259]
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), lens, scale)
    emin = [int(pl[pl > 0].min()) for pl in (planes[1], planes[3])]
    for max_len in (S, S_max):        # one workgroup of eight wavefronts a sequence (4 bits, 16-bit I/O, up to 8 heads), splits
        got = kvbfp.decode_attention(cache, q.cuda(), max_len, scale,
                                     seq_len_dev=torch.tensor(lens, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        assert bool(torch.isfinite(got).all())
        assert_attention_close(got, want, dtype, "%s n=%d p=%d shifts k %d v %d q %d (smallest exponent bytes %s) max_len %d" % (
            DT_NAME[dtype], n, p, k_shift, v_shift, q_shift, emin, max_len))


@pytest.mark.parametrize("dtype,n,p", FAMILIES)
@pytest.mark.parametrize("v_shift", [-100, -120, 110])
def test_values_at_the_ends_of_the_range(dtype, n, p, v_shift):
    if dtype == torch.float16:
        v_shift = {-100: -8, -120: -12, 110: 2}[v_shift]       # fp16 inputs: the ends of ITS range
    _run(dtype, n, p, 0, v_shift, 0)


@pytest.mark.parametrize("dtype,n,p", FAMILIES)
@pytest.mark.parametrize("k_shift", [-100, 100])
def test_keys_at_the_ends_of_the_range_with_the_matching_softmax_scale(dtype, n, p, k_shift):
    if dtype == torch.float16:
        k_shift = -10 if k_shift < 0 else 4
    _run(dtype, n, p, k_shift, 0, 0)


@pytest.mark.parametrize("dtype,n,p", FAMILIES)
def test_tiny_keys_with_an_ordinary_softmax_scale_give_the_plain_average(dtype, n, p):
    # scores of the order 2^-120: the softmax is flat and the output is the mean of the cached values
    _run(dtype, n, p, -10 if dtype == torch.float16 else -120, 0, 0, compensate=False)


@pytest.mark.parametrize("dtype,n,p", FAMILIES)
@pytest.mark.parametrize("q_shift", [-90, 90])
def test_queries_at_the_ends_of_the_range_with_the_matching_softmax_scale(dtype, n, p, q_shift):
    if dtype == torch.float16:
        q_shift = -10 if q_shift < 0 else 4
    _run(dtype, n, p, 0, 0, q_shift)


@pytest.mark.parametrize("G", [12, 40])           # the passes for 9 to 32 heads and for more
@pytest.mark.parametrize("dtype,n,p", [f for f in FAMILIES if f[0] != torch.float32])
@pytest.mark.parametrize("which,shift", [("k", -100), ("k", 100), ("q", -90), ("q", 90), ("v", -100), ("v", -120), ("v", 110)])
def test_many_heads_at_the_ends_of_the_range(dtype, n, p, which, shift, G):
    if dtype == torch.float16:
        shift = {"k": {-100: -10, 100: 4}, "q": {-90: -10, 90: 4}, "v": {-100: -8, -120: -12, 110: 2}}[which][shift]
    _run(dtype, n, p, shift if which == "k" else 0, shift if which == "v" else 0, shift if which == "q" else 0, G=G)


@pytest.mark.parametrize("B,Hkv,S,splits", [(2, 2, 1500, 6), (3, 64, 2400, 4), (4, 64, 3100, 3), (6, 64, 700, 2), (2, 2, 1024, 0), (2, 2, 700, 0), (2, 2, 300, 0)])
def test_sums_beyond_the_range_are_infinite_whatever_the_number_of_splits(B, Hkv, S, splits):
    # the value sums of a split leave fp32 before the division by the normaliser: an infinity, and no NaN from a
    # split that is not there (0: one workgroup, which writes the output itself)
    v = torch.full((B, S, Hkv, D), 2.0 ** 125, dtype=torch.bfloat16, device="cuda")
    k = synth.kv_rows(B, S, Hkv, D, "bf16", synth.outlier_gains(5, 0, Hkv, D), 5, 2, "cuda")
    q = synth.queries(B, 4 * Hkv, D, "bf16", 5, 4)
    cache = gpu_cache(k, v, 32, 4, S)
    ws = torch.zeros(kvbfp.decode_workspace_bytes(cache.layout, 4 * Hkv, S), dtype=torch.uint8, device="cuda")
    got = kvbfp.decode_attention(cache, q.cuda(), S, 1e-3, workspace=ws)
    torch.cuda.synchronize()
    assert bool(torch.isposinf(got).all())
    heads = B * 4 * Hkv                              # rows of partial results: an infinity and no zero in each that was written
    assert int((ws.view(torch.float32)[:heads * splits * D].view(-1, D)[:, 0] != 0).sum()) == heads * splits
    assert bool(ws.any()) == (splits > 0)
