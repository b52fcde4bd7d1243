"""Many (virtual) query heads per kv-head: the pass that decodes cached rows once to bf16 and multiplies whole
matrix-core tiles with them (decode_wide.hip), against the oracle at the edges of its tiles of 32 heads and of 64 and
128 tokens, over regions and pages, with queries as given and cast to BFP."""
import numpy as np
import pytest
import torch

from oracle import kvbfp_oracle as O
from paper_2403_20137_amd import kvbfp, synth
from test_gpu_paged import fill_both
from util import assert_attention_close, assert_planes_equal, dev_i32, gpu_cache, oracle_cache

pytestmark = pytest.mark.gpu
D = 128
DT = {"f16": torch.float16, "bf16": torch.bfloat16}
LENS = [517, 1, 64, 129, 255]          # below, at and above the 64- and 128-token tiles, and a single token


def _inputs(dt, Hkv, S, B, seed, heads):
    kg, vg = synth.outlier_gains(seed, 0, Hkv, D), synth.outlier_gains(seed, 1, Hkv, D)
    k = synth.kv_rows(B, S, Hkv, D, dt, kg, seed, 2)
    v = synth.kv_rows(B, S, Hkv, D, dt, vg, seed, 3)
    q = synth.queries(B, heads, D, dt, seed, 4)
    pk = O.calibrate_perm(synth.to_f32_numpy(synth.kv_rows(1, 32, Hkv, D, dt, kg, seed, 5)[0]))
    pv = O.calibrate_perm(synth.to_f32_numpy(synth.kv_rows(1, 32, Hkv, D, dt, vg, seed, 6)[0]))
    return k, v, q, pk, pv


@pytest.mark.parametrize("dt,p,n,G,Tq,qbits,page", [
    ("bf16", 4, 32, 9, 1, 0, 0),
    ("f16", 8, 16, 16, 1, 0, 0),
    ("bf16", 4, 32, 17, 1, 0, 0),       # one group of 32 heads, mostly unused
    ("bf16", 4, 16, 4, 8, 0, 16),       # exactly 32
    ("f16", 4, 32, 11, 3, 0, 0),        # 33: two groups
    ("bf16", 4, 64, 8, 8, 8, 64),       # exactly 64
    ("f16", 8, 16, 13, 5, 0, 16),       # 65: three of four groups
    ("bf16", 8, 32, 32, 4, 8, 0),       # exactly 128
    ("bf16", 4, 128, 43, 3, 4, 0),      # 129: two workgroups
    ("f16", 4, 16, 20, 13, 8, 32),      # 260: three workgroups, fp16 query cast to BFP
    ("f16", 8, 64, 33, 4, 0, 256),
])
def test_against_the_oracle(dt, p, n, G, Tq, qbits, page):
    B, Hkv, S = len(LENS), 2, max(LENS)
    k, v, q, pk, pv = _inputs(dt, Hkv, S, B, 40 + G + p, Hkv * G * Tq)
    q = q.view(B, Tq, Hkv * G, D).contiguous()
    scale = float(np.float32(-0.07 if qbits == 4 else 0.09))          # the sign of the scale travels with the query
    lens = dev_i32(np.asarray(LENS))
    kw = dict(seq_len_dev=lens, perm_k=dev_i32(pk), perm_v=dev_i32(pv), q_mant_bits=qbits)
    if page:
        pages = -(-S // page)
        pool, table, planes = fill_both(k, v, n, p, page, pages, LENS, pk, pv, 7)
        got = kvbfp.decode_attention_multi_paged(pool, table, q.cuda(), S, scale, **kw)
    else:
        planes = oracle_cache(k, v, n, p, S, 0, pk, pv)
        cache = gpu_cache(k.cuda(), v.cuda(), n, p, S, perm_k=pk, perm_v=pv)
        got = kvbfp.decode_attention_multi(cache, q.cuda(), S, scale, **kw)
    torch.cuda.synchronize()
    for i in range(Tq):
        seen = [max(l - (Tq - 1 - i), 0) for l in LENS]
        want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q[:, i]), seen, scale, pk, pv, q_mant_bits=qbits)
        assert_attention_close(got[:, i], want, DT[dt], "G=%d Tq=%d p=%d n=%d page=%d, token %d" % (G, Tq, p, n, page, i))


@pytest.mark.parametrize("G", [12, 40, 150])       # cast inside the pass (one workgroup has all heads) and ahead of it
@pytest.mark.parametrize("lens", [[300, 1, 65], [128, 0, 129]])
def test_append_equals_two_calls(G, lens):
    B, Hkv, S, n, p = len(lens), 2, 320, 32, 4
    k, v, q, pk, pv = _inputs("bf16", Hkv, S, B, 90 + G, Hkv * G)
    kn, vn = (synth.kv_rows(B, 1, Hkv, D, "bf16", synth.outlier_gains(5, 0, Hkv, D), 5, t).cuda() for t in (7, 8))
    kw = dict(seq_len_dev=dev_i32(np.asarray(lens)), perm_k=dev_i32(pk), perm_v=dev_i32(pv))
    one, two = (gpu_cache(k.cuda(), v.cuda(), n, p, S, perm_k=pk, perm_v=pv) for _ in range(2))
    kvbfp.quantize_append(two, kn, vn, pos_dev=kw["seq_len_dev"] - 1, perm_k=kw["perm_k"], perm_v=kw["perm_v"])
    b = kvbfp.decode_attention(two, q.cuda(), S, 0.1, **kw)
    a = kvbfp.append_decode_attention(one, kn, vn, q.cuda(), S, 0.1, **kw)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and all(torch.equal(x, y) for x, y in zip(one.planes(), two.planes()))


@pytest.mark.parametrize("k_shift,q_shift", [(-100, 0), (100, 0), (0, -90), (0, 90)])
@pytest.mark.parametrize("p", [4, 8])
def test_ends_of_the_range(p, k_shift, q_shift):
    B, Hkv, G, S, n = 2, 1, 33, 300, 32
    k, v, q, _, _ = _inputs("bf16", Hkv, S, B, 3, Hkv * G)
    k, q = (k.float() * 2.0 ** k_shift).bfloat16(), (q.float() * 2.0 ** q_shift).bfloat16()
    planes = oracle_cache(k, v, n, p, S, 0)
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    assert_planes_equal(cache, planes)
    scale = float(np.float32(0.09) * np.float32(2.0 ** -(k_shift + q_shift)))
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert_attention_close(got, O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S, S], scale), torch.bfloat16)


@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("n", [16, 32])
@pytest.mark.parametrize("which,byte", [("k", 255), ("v", 254), ("k", 1), ("v", 1), ("v", 2)])
def test_every_exponent_byte(p, n, which, byte):
    """Blocks with the first and last exponent bytes next to ordinary ones, written into the planes as they are."""
    B, Hkv, G, S = 1, 1, 33, 200
    k, v, q, _, _ = _inputs("bf16", Hkv, S, B, 3, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0)
    scale = float(np.float32(0.09))
    mant, exps = (planes[0], planes[1]) if which == "k" else (planes[2], planes[3])
    if byte > 200:      # block 0 of some tokens; as keys against a query that is tiny there
        exps[0, 0, [150] if which == "v" else slice(None, None, 3), 0] = byte
        if which == "k":
            q = q.float()
            q[..., :n] *= 2.0 ** -126
            q = q.bfloat16()
    elif which == "k":  # all blocks of all keys at the lowest bytes, the scale to match
        exps[:] = byte + (np.arange(exps.size).reshape(exps.shape) % 2)
        q, scale = (q.float() * 2.0 ** 60).bfloat16(), float(np.float32(2.0 ** 60))
    else:               # values: the output is as small as they are, compared after scaling up
        exps[:] = byte
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w))
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S], scale)
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(got).all()) and np.isfinite(want).all()
    if which == "v" and byte < 200:
        # bf16 outputs below 2^-126 have an absolute step of 2^-133
        diff = np.abs(got.cpu().double().numpy() - want)
        assert (diff <= 2.0 ** -134 + 2.0 ** -8 * np.abs(want)).all(), diff.max()
    else:
        assert_attention_close(got, want, torch.bfloat16, "%s %d" % (which, byte))


@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("n", [16, 32, 64, 128])
@pytest.mark.parametrize("byte,beside", [(1, None), (2, None), (1, 20), (3, None)])
def test_keys_with_the_smallest_exponent_bytes_up_to_32_heads(p, n, byte, beside):
    """Keys are exact at every byte a finite row can have, as in the passes for up to 8 heads: with the scale to match, the
    scores come out as anywhere else.  beside: the first 16 tokens of every 40 hold larger ones."""
    B, Hkv, G, S = 1, 1, 12, 200
    k, v, q, _, _ = _inputs("bf16", Hkv, S, B, 3, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0)
    planes[1][:] = byte + (np.arange(planes[1].size).reshape(planes[1].shape) % 2)
    if beside:
        planes[1][:, :, np.arange(S) % 40 < 16] = beside
    q, scale = (q.float() * 2.0 ** 60).bfloat16(), float(np.float32(2.0 ** (60 if not beside else 44)))
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w))
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert_attention_close(got, O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S], scale), torch.bfloat16)


@pytest.mark.parametrize("p,top", [(4, 254), (4, 253), (4, 252), (8, 251), (8, 250), (8, 249)])
@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_keys_with_the_largest_exponent_bytes_up_to_32_heads(p, n, top):
    """Every third token's rows at the last bytes the pass takes and around them, the others 2^20 smaller."""
    B, Hkv, G, S = 1, 1, 12, 200
    k, v, q, _, _ = _inputs("bf16", Hkv, S, B, 3, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0)
    planes[1][:] = top - 20
    planes[1][:, :, ::3] = top
    q, scale = (q.float() * 2.0 ** -60).bfloat16(), float(np.float32(2.0 ** -(top - 127 - 60)) * np.float32(0.05))
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w))
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert_attention_close(got, O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S], scale), torch.bfloat16)


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("p,n", [(4, 16), (4, 32), (8, 32)])
@pytest.mark.parametrize("G", [40, 100, 130])
def test_partial_results_above_32_heads_are_fp32(dt, p, n, G):
    """More than 32 heads: probabilities keep their 24 bits.  The workspace holds the partial results in fp32; merged here
    in 64 bits they are as far from the oracle as fp32 sums over the scores' rounding are: 2100 products of weights
    whose base-2 scores of magnitude up to 16 carry 2^-24 of it each, 16 * 2^-24 = 1e-6 times a few for the sum of
    128 products behind a score."""
    B, S, Hkv = 2, 2100, 1
    k, v, q, pk, _ = _inputs(dt, Hkv, S, B, 5, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0, pk, None)
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S, perm_k=pk)
    scale, Hq = float(np.float32(D ** -0.5)), Hkv * G
    need = kvbfp.decode_workspace_bytes(cache.layout, Hq, S)
    splits = need // (B * Hq * (D + 2) * 4)
    ws = torch.zeros((need,), dtype=torch.uint8, device="cuda")
    kvbfp.decode_attention(cache, q.cuda(), S, scale, perm_k=dev_i32(pk), workspace=ws)
    torch.cuda.synchronize()
    f = ws.view(torch.float32).cpu().double().numpy()
    po, ml = f[:B * Hq * splits * D].reshape(B, Hq, splits, D), f[B * Hq * splits * D:].reshape(B, Hq, splits, 2)
    assert (ml[..., 1] > 0).all()
    w = np.exp2(ml[..., 0] - ml[..., 0].max(axis=-1, keepdims=True))
    merged = (w[..., None] * po).sum(axis=2) / (w * ml[..., 1]).sum(axis=-1)[..., None]
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S, S], scale, pk, None)
    err = np.linalg.norm(merged - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() <= 6e-6 and err.mean() <= 6e-7, (err.max(), err.mean())


@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("dt,q_exp,s_exp", [("bf16", -120, -12), ("f16", -12, -120), ("bf16", -60, -72)])
def test_query_far_below_one_times_a_small_scale(p, dt, q_exp, s_exp):
    """q * softmax_scale around 2^-132, where fp32 itself is short of bits, against keys around 2^124: the scores count."""
    B, Hkv, G, S, n = 1, 1, 40, 300, 32
    gen = torch.Generator().manual_seed(8)
    k, v = (torch.randn(B, S, Hkv, D, generator=gen) * f for f in (2.0 ** 124, 1.0))
    k, v = k.clamp(-2.0 ** 126, 2.0 ** 126).bfloat16(), v.bfloat16()
    q = (torch.randn(B, Hkv * G, D, generator=gen) * 2.0 ** q_exp).to(DT[dt])
    planes = oracle_cache(k, v, n, p, S, 0)
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    scale = float(np.float32(2.0 ** s_exp))
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S], scale)
    flat = O.decode_attention(*planes, D, n, p, 0 * synth.to_f32_numpy(q), [S], scale)
    assert np.linalg.norm(want - flat) > 0.02 * np.linalg.norm(want)
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert_attention_close(got, want, DT[dt])


@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("G", [40, 100])
@pytest.mark.parametrize("which", ["k", "v"])
@pytest.mark.parametrize("top,byte", [(255, 1), (255, 6), (252, 2), (252, 7)])
def test_largest_exponent_bytes_beside_the_smallest(p, n, G, which, top, byte):
    """Block 0 of two tokens of every 16 holds the largest numbers (code 1 or 17, so that their mean stays in fp32), all
    other blocks the smallest: every block is exact whatever stands beside it."""
    B, Hkv, S = 1, 1, 200
    k, v, q, _, _ = _inputs("bf16", Hkv, S, B, 3, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0)
    mant, exps = (planes[0], planes[1]) if which == "k" else (planes[2], planes[3])
    exps[:] = byte
    for t in (0, 5):
        exps[0, 0, t::16, 0] = top
        mant[0, 0, t::16, :n * p // 8] = 0x11
    scale = float(np.float32(0.09))
    if which == "k":    # what is large meets a query of zeros there, what is small one that is large
        q = q.float() * 2.0 ** 60
        q[..., :n] = 0
        q, scale = q.bfloat16(), float(np.float32(2.0 ** (60 - byte)))
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w))
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S], scale)
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert np.isfinite(want).all() and np.abs(want).max() < 2.0 ** 127
    if which == "k":
        assert_attention_close(got, want, torch.bfloat16)
        return
    # by element: bf16 outputs below 2^-126 have an absolute step of 2^-133
    diff = np.abs(got.cpu().double().numpy() - want)
    slack = np.empty_like(diff)
    for part in (slice(0, n), slice(n, D)):
        slack[..., part] = 3e-4 * np.abs(want[..., part]).max(axis=-1, keepdims=True)
    assert (diff <= 2.0 ** -134 + 2.0 ** -8 * np.abs(want) + slack).all(), (diff / np.abs(want)).max()


@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("n", [16, 32, 64, 128])
@pytest.mark.parametrize("byte", [1, 2, 3, 254])
def test_values_at_the_ends_of_the_exponent_bytes_up_to_32_heads(p, n, byte):
    """Bytes 3 to 254 (8-bit: 251) are exact; 1 and 2 are off by less than 2^-126 an element, as documented."""
    B, Hkv, G, S = 1, 1, 12, 200
    k, v, q, _, _ = _inputs("bf16", Hkv, S, B, 3, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0)
    if byte > 200:
        planes[3][0, 0, 150, 0] = byte if p == 4 else 251
    else:
        planes[3][:] = byte
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w))
    scale = float(np.float32(0.09))
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), [S], scale)
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    if byte > 200:
        assert_attention_close(got, want, torch.bfloat16)
    else:
        diff = np.abs(got.cpu().double().numpy() - want)
        assert (diff <= (2.0 ** -126 if byte < 3 else 0) + 2.0 ** -134 + 2.0 ** -8 * np.abs(want)).all(), diff.max()


@pytest.mark.parametrize("G", [12, 40])
def test_query_and_output_at_any_address(G):
    B, Hkv, S = 1, 1, 200
    k, v, q, pk, pv = _inputs("bf16", Hkv, S, B, 11, G)
    cache = gpu_cache(k.cuda(), v.cuda(), 32, 4, S)
    want = kvbfp.decode_attention(cache, q.cuda(), S, 0.1, perm_v=dev_i32(pv))
    shifted = torch.zeros(q.numel() + 1, dtype=q.dtype, device="cuda")
    shifted[1:] = q.cuda().flatten()
    out = torch.zeros(q.numel() + 1, dtype=q.dtype, device="cuda")
    got = kvbfp.decode_attention(cache, shifted[1:].view(q.shape), S, 0.1, perm_v=dev_i32(pv), out=out[1:].view(q.shape))
    torch.cuda.synchronize()
    assert torch.equal(got, want) and float(out[0]) == 0.0


@pytest.mark.parametrize("dt,p,n,G", [("bf16", 4, 32, 33), ("f16", 4, 16, 70), ("bf16", 8, 16, 33), ("f16", 8, 64, 70)])
def test_exponents_that_leave_the_range_of_the_first_tile(dt, p, n, G):
    """Two workgroups a sequence, four tiles each: exponents far from those of a workgroup's first tile in a later one.  Block 0 (and the keys)
    of one sequence each: nothing; one value 2^30 above; 2^40 below; 2^40 below from the start on, then as it was; zero rows at
    the start; one value 2^10 above in the last token; keys at the smallest byte; up by 2^6 and down by 2^24, the last that fit."""
    B, Hkv, S = 64, 4, 450
    k, v, q, _, _ = _inputs(dt, Hkv, S, B, 17 + G, Hkv * G)
    planes = oracle_cache(k, v, n, p, S, 0)
    ke, ve = planes[1], planes[3]
    for b in range(B):
        t = 128 + 64 * (b // 8 % 4) + b % 16               # second to fifth tile
        e = ve[b, ..., 0].astype(np.int64)
        kind = b % 8
        if kind == 1: e[:, t] += 30
        elif kind == 2: e[:, t] -= 40
        elif kind == 3: e[:, :t] -= 40
        elif kind == 4: ve[b, :, :t], planes[2][b, :, :t] = 0, 0
        elif kind == 5: e[:, S - 1] += 10
        elif kind == 6: ke[b, :, t:t + 16] = 1
        elif kind == 7:
            e[:, t] += 6
            e[:, t + 9] -= 24
        if kind != 4:
            ve[b, ..., 0] = e
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w))
    scale = float(np.float32(0.02))
    want = O.decode_attention(*(np.ascontiguousarray(x[:, 1:2]) for x in planes), D, n, p, synth.to_f32_numpy(q[:, G:2 * G]), [S] * B, scale)   # one kv-head
    if dt == "f16":                                        # block 0 of the values out of its range: compared as it is stored
        want = np.where(np.abs(want) < 65520, want, np.inf * np.sign(want))
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)[:, G:2 * G]
    torch.cuda.synchronize()
    for part in (slice(0, n), slice(n, D)):                # apart: what is large in block 0 says nothing about the others
        g, w = got[..., part], want[..., part]
        fits = np.isfinite(w).all(axis=-1)
        assert bool((torch.isinf(g).cpu() == torch.from_numpy(np.isinf(w))).all())
        for b in range(B):
            if fits[b].any():
                assert_attention_close(g[b, fits[b]], w[b, fits[b]], DT[dt], "sequence %d" % b)


@pytest.mark.parametrize("p,top", [(4, 240), (8, 240), (4, 201)])
@pytest.mark.parametrize("G", [12, 40])
def test_sums_of_large_values_while_the_scores_rise(p, top, G):
    """4096 tokens of one weight, near what their sum can be in fp32, behind some whose scores are 3.5 powers of two lower: the
    reference of the sums may not be the one of those.  (Byte 201 is the first on that path; its sums would fit either way.  12 heads
    with 8 bits rescale at every new maximum.)"""
    B, Hkv, S, n = 64, 4, 4096, 32
    layout = kvbfp.make_layout(D, n, p, Hkv, B, S)
    cache = kvbfp.alloc_cache(layout, "cuda", fill=0)
    one, seven = (0x11, 0x77) if p == 4 else (0x10, 0x70)
    cache.k_mant[:, :, 256:] = one
    cache.k_exp[:] = 129
    cache.v_mant[:] = seven
    cache.v_exp[:] = top
    key = 1.0 if p == 4 else 2.0 ** -4 * 16             # a code times 2^(129 - 127 - (p - 2))
    value = 7.0 * 2.0 ** (top - 129) if p == 4 else 112.0 * 2.0 ** (top - 133)
    assert S * value < 2.0 ** 128
    q = torch.ones((B, Hkv * G, D), dtype=torch.bfloat16, device="cuda")
    got = kvbfp.decode_attention(cache, q, S, float(np.float32(3.5 / (D * key * np.log2(np.e)))))
    torch.cuda.synchronize()
    assert bool((got.double() / value - 1).abs().max() < 2.0 ** -8)


@pytest.mark.parametrize("heavy", ["zero row", "zero channels", "small blocks"])
@pytest.mark.parametrize("gap", [20.3, 30.7, 40.2])
@pytest.mark.parametrize("p,n,G", [(4, 16, 40), (4, 32, 100), (8, 32, 40), (8, 64, 100)])
def test_light_tokens_beside_a_heavy_one_above_32_heads(p, n, G, gap, heavy):
    """One token's score is `gap` powers of two above the others and its value row holds nothing, nothing in every other channel,
    or blocks 2^24 below the others': what the light tokens sum to there keeps the bits of an fp32 sum.  The one split's
    partial results, compared by channel with what weights off by 40 * 2^-24 times a few (the rounding of a score) make of
    the sum of the magnitudes."""
    B, Hkv, S = 128, 4, 300                             # 512 units: one split
    rng = np.random.default_rng(int(gap * 10) + p + G)
    ms, es = O.plane_shapes(1, 1, D, n, p, S)
    km, ke, vm, ve = np.zeros(ms, np.uint8), np.full(es, 127, np.uint8), np.zeros(ms, np.uint8), np.full(es, 127, np.uint8)
    one = 0x11 if p == 4 else 0x10
    km[0, 0, :, :2] = rng.integers(0, 256, (S, 2)) & (0x33 if p == 4 else 0x1F)      # light scores a little apart
    vm[:] = rng.integers(0, 256, ms)
    ve[:] = 127 + rng.integers(-3, 4, es)
    km[0, 0, 3] = one
    if heavy == "zero row":
        vm[0, 0, 3], ve[0, 0, 3] = 0, 0
    elif heavy == "zero channels":
        if p == 4:
            vm[0, 0, 3] &= 0xF0
        else:
            vm[0, 0, 3, ::2] = 0
    else:
        vm[0, 0, 3], ve[0, 0, 3] = one, 127 - 24
    planes = [km, ke, vm, ve]
    cache = kvbfp.alloc_cache(kvbfp.make_layout(D, n, p, Hkv, B, S), "cuda", fill=0)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w).expand(t.shape))
    q = (1 + 0.1 * torch.rand((1, Hkv * G, D), generator=torch.Generator().manual_seed(3))).bfloat16()
    scale = float(np.float32(gap / (1.05 * D * 0.25 * np.log2(np.e))))           # a code of one is 2^-2
    Hq = Hkv * G
    ws = torch.zeros((max(kvbfp.decode_workspace_bytes(cache.layout, Hq, S), B * Hq * (D + 2) * 4),), dtype=torch.uint8, device="cuda")
    kvbfp.decode_attention(cache, q.expand(B, Hq, D).contiguous().cuda(), S, scale, workspace=ws)
    torch.cuda.synchronize()
    f = ws.view(torch.float32)
    po, ml = f[:B * Hq * D].view(B, Hq, D), f[B * Hq * D:B * Hq * (D + 2)].view(B, Hq, 2)
    assert torch.equal(po[:1].expand_as(po)[..., :G, :], po[..., :G, :])
    got = (po[-1, :G].double() / ml[-1, :G, 1:].double()).cpu().numpy()
    qf = synth.to_f32_numpy(q[:, :G])
    want = O.decode_attention(*planes, D, n, p, qf, [S], scale)[0]
    size = O.decode_attention(km, ke, vm & (0x77 if p == 4 else 0x7F), ve, D, n, p, qf, [S], scale)[0]
    err = np.abs(got - want) / np.where(size > 0, size, 1)
    assert err.max() <= 2e-5, (err.max(), np.unravel_index(err.argmax(), err.shape))


# (tiles of (score in units of 3.5 powers of two, large values) per quarter of a tile; splits)
@pytest.mark.parametrize("name,tiles,splits", [
    ("large values behind a rise", [[(0, 0)] * 4, [(1, 0)] * 4, [(0, 1)] * 4], 1),
    ("large values ahead of a rise", [[(0, 1)] * 4, [(1, 0)] * 4], 1),
    ("a rise in another wavefront", [[(0, 1)] * 3 + [(0, 0)], [(-7, 0)] * 3 + [(1, 0)]], 1),
    ("a rise in another split", [[(0, 1)] * 4] * 3 + [[(0, 0)] * 4] + [[(-7, 0)] * 4] * 11 + [[(1, 0)] * 4], 4),
])
@pytest.mark.parametrize("p,G", [(4, 12), (8, 12), (4, 40), (8, 40), (4, 100), (8, 100)])
def test_sums_of_large_values_where_the_scores_rose(p, G, name, tiles, splits):
    """Sums of values near the end of fp32 relative to the largest score so far fit; relative to one 3.5 powers of two lower they do
    not, in a wavefront, in the merge of its workgroup or in that of the splits."""
    TT = 128 if G <= 32 else 64
    B, Hkv, S, n = 512 // splits // 4, 4, TT * len(tiles), 32
    # as many as a wavefront (where all four hold values, its sum alone fits) or a split has: 7 2^(byte - 129) each, below 2^128 in all
    together = TT if splits > 1 or G > 64 else 32
    byte = 254 - int(np.log2(together))
    ms, es = O.plane_shapes(1, 1, D, n, p, S)
    km, ke, vm, ve = np.zeros(ms, np.uint8), np.full(es, 127, np.uint8), np.zeros(ms, np.uint8), np.full(es, 127, np.uint8)
    codes = {0: 0, 1: 0x11, -7: 0xFF} if p == 4 else {0: 0, 1: 0x10, -7: 0xF0}
    for i, tile in enumerate(tiles):
        for j, (score, large) in enumerate(tile):
            part = slice(i * TT + j * TT // 4, i * TT + (j + 1) * TT // 4)
            km[0, 0, part] = codes[score]
            vm[0, 0, part] = 0x77 if p == 4 else 0x70
            ve[0, 0, part] = byte if large else 127
    planes = [km, ke, vm, ve]
    cache = kvbfp.alloc_cache(kvbfp.make_layout(D, n, p, Hkv, B, S), "cuda", fill=0)
    for t, w in zip(cache.planes(), planes):
        t.copy_(torch.from_numpy(w).expand(t.shape))
    q = torch.ones((B, Hkv * G, D), dtype=torch.bfloat16)
    scale = float(np.float32(3.5 / (D * 0.25 * np.log2(np.e))))                  # a code of one is 2^-2
    got = kvbfp.decode_attention(cache, q.cuda(), S, scale)
    torch.cuda.synchronize()
    want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q[:1, :1]), [S], scale)[0, 0, 0]
    assert 2.0 ** 100 < want < 2.0 ** 127
    assert bool((got.double() / want - 1).abs().max() < 2.0 ** -8), (name, float(got.double().max()), want)
