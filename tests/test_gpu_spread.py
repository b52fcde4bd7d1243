"""Sequences of different lengths: the workgroups of a kv-head shared out by the lengths (decode_spans.h), for every split
pass that does so, against the oracle.  Batch and head counts and the longest sequence are such that its splits would have
several tiles each (7 and more with 4-bit mantissas and 16-bit I/O, 3 and more in the other passes), where sharing out applies;
sizes below that are among them too."""
import numpy as np
import pytest
import torch

from test_gpu_attention import make_small, run_both
from test_gpu_rope_at_read import run_both as run_rope
from util import assert_attention_close, dev_i32, gpu_cache, oracle_cache, rel_l2_per_head
from oracle import kvbfp_oracle as O
from paper_2403_20137_amd import kvbfp, synth

pytestmark = pytest.mark.gpu
D = 128


def _lens(B, S, seed, long_only=False):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 100, B) if long_only else np.exp(rng.uniform(0, np.log(S), B)).astype(np.int64)
    lens[rng.integers(B)] = S
    if B > 3:
        lens[np.flatnonzero(lens != S)[0]] = 0
    return [int(x) for x in lens]


@pytest.mark.parametrize("dtype,p,n,G,B,Hkv,S", [
    (torch.bfloat16, 4, 32, 1, 70, 8, 1100),      # not shared out
    (torch.bfloat16, 4, 32, 1, 70, 8, 4200),      # more than 64 sequences, two splits, 17 tiles; LDS pipeline
    (torch.bfloat16, 4, 64, 8, 64, 8, 3700),      # exactly 64
    (torch.bfloat16, 4, 32, 2, 300, 1, 6000),     # more than 256 (three splits)
    (torch.bfloat16, 4, 32, 2, 767, 1, 3700),     # as many as two splits allow
    (torch.float16, 8, 16, 1, 40, 8, 1100),       # 8-bit pipeline
    (torch.float16, 8, 64, 5, 25, 8, 2100),
    (torch.float32, 4, 16, 1, 40, 8, 900),        # register-staged passes
    (torch.float32, 8, 32, 1, 40, 8, 900),
    (torch.float32, 8, 32, 1, 65, 4, 2000),
    (torch.float32, 4, 32, 12, 24, 8, 2000),      # two launches over head subsets
    (torch.bfloat16, 4, 32, 12, 24, 8, 900),      # 9 to 32 heads, tiles of 128
    (torch.bfloat16, 8, 128, 20, 24, 8, 900),
    (torch.bfloat16, 4, 16, 40, 12, 8, 700),      # more heads, tiles of 64: not shared out
    (torch.bfloat16, 4, 16, 40, 12, 8, 2000),
    (torch.float16, 8, 32, 150, 12, 8, 1000),     # two workgroups per split
    (torch.bfloat16, 4, 32, 4, 3, 64, 1500),      # three sequences
    (torch.bfloat16, 4, 32, 4, 3, 64, 9500),
])
def test_against_the_oracle(dtype, p, n, G, B, Hkv, S):
    lens = _lens(B, S, B)
    k, v, q, pk, pv = make_small(dtype, B=B, S=S, Hkv=Hkv, G=G, seed=500 + B)
    got, want = run_both(k, v, q, n, p, lens, 128 ** -0.5, pk, pv)
    assert_attention_close(got, want, dtype, "lens %s" % lens)


def test_one_long_sequence_among_many_short_ones():
    # it gets more places than the combine pass merges at a time (32)
    B, S = 100, 12000
    lens = _lens(B, S, 3, long_only=True)
    k, v, q, pk, pv = make_small(torch.bfloat16, B=B, S=S, Hkv=2, G=4, seed=600)
    got, want = run_both(k, v, q, 32, 4, lens, 128 ** -0.5, pk, pv)
    assert_attention_close(got, want, torch.bfloat16)


def test_more_than_32_splits():
    B, S = 2, 13000                              # 2 x 8 units: 48 splits; the 32-channel combine
    k, v, q, pk, pv = make_small(torch.bfloat16, B=B, S=S, Hkv=8, G=1, seed=610)
    got, want = run_both(k, v, q, 32, 4, [S, 300], 128 ** -0.5, pk, pv)
    assert_attention_close(got, want, torch.bfloat16)


@pytest.mark.parametrize("dtype,p,B,Hkv,G,S", [
    (torch.float32, 4, 4, 2, 1, 60000),          # 96 splits, 235 tiles: the 32-channel form of the combine pass
    (torch.bfloat16, 8, 4, 2, 40, 30000),        # 64 splits, 469 tiles of 64 tokens, 320 heads: the 128-channel form
    (torch.bfloat16, 4, 3, 4, 20, 33000),        # 42 splits, 258 tiles of 128
])
def test_shared_out_among_more_than_32_splits(dtype, p, B, Hkv, G, S):
    k, v, q, pk, pv = make_small(dtype, B=B, S=S, Hkv=Hkv, G=G, seed=611)
    got, want = run_both(k, v, q, 32, p, [S, 300, 1, 2000][:B], 128 ** -0.5, pk, pv)
    assert_attention_close(got, want, dtype)


@pytest.mark.parametrize("dtype,p,n,G,Tq,qbits,page,B,S", [
    (torch.bfloat16, 4, 32, 4, 1, 0, 16, 40, 4096),       # LDS pipeline
    (torch.bfloat16, 4, 32, 8, 1, 8, 256, 40, 4096),      # its two head groups
    (torch.float16, 8, 32, 2, 1, 8, 32, 25, 2100),        # integer score product
    (torch.float16, 8, 16, 1, 3, 0, 64, 25, 2100),        # three query tokens
    (torch.float32, 4, 16, 2, 2, 0, 16, 40, 2000),        # register-staged passes
    (torch.float32, 8, 64, 1, 1, 4, 128, 25, 2100),
    (torch.float32, 4, 32, 3, 5, 0, 32, 40, 2000),        # two launches
    (torch.bfloat16, 4, 32, 4, 5, 0, 16, 24, 900),        # 20 heads
    (torch.float16, 8, 64, 3, 4, 8, 64, 70, 1500),        # 12, one split of 70 x 8: not shared out
    (torch.float16, 4, 16, 5, 9, 0, 16, 12, 2000),        # 45
    (torch.bfloat16, 8, 32, 4, 40, 0, 256, 12, 1000),     # 160
])
def test_pages_query_tokens_and_query_cast(dtype, p, n, G, Tq, qbits, page, B, S):
    Hkv = 8
    lens = _lens(B, S, B + S)
    k, v, q, pk, pv = make_small(dtype, B=B, S=S, Hkv=Hkv, G=G * Tq, seed=650 + Tq)
    q = q.view(B, Tq, Hkv * G, 128).contiguous()
    kw = dict(seq_len_dev=dev_i32(np.asarray(lens)), perm_k=dev_i32(pk), perm_v=dev_i32(pv), q_mant_bits=qbits)
    scale = float(np.float32(0.09))
    # the bytes of the pool are those of the region (compared with the oracle elsewhere), page by page
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, -(-S // page) * page, perm_k=pk, perm_v=pv)
    per_seq = -(-S // page)
    table = np.random.default_rng(B).permutation(B * per_seq).reshape(B, per_seq).astype(np.int32)
    pool = kvbfp.alloc_cache(kvbfp.make_layout(128, n, p, Hkv, B * per_seq, page), "cuda", fill=0)
    for dst, src in zip(pool.planes(), cache.planes()):
        rows = src.view(B, Hkv, per_seq, page, -1).transpose(1, 2).reshape(B * per_seq, Hkv, page, -1)
        dst[torch.as_tensor(table.reshape(-1), device="cuda").long()] = rows.reshape(dst.shape)
    got = kvbfp.decode_attention_multi_paged(pool, dev_i32(table), q.cuda(), S, scale, **kw)
    flat = kvbfp.decode_attention_multi(cache, q.cuda(), S, scale, **kw)
    torch.cuda.synchronize()
    assert torch.equal(got, flat)
    planes = [x.cpu().numpy() for x in cache.planes()]
    for i in {0, Tq - 1}:
        seen = [max(l - (Tq - 1 - i), 0) for l in lens]
        want = O.decode_attention(*planes, 128, n, p, synth.to_f32_numpy(q[:, i]), seen, scale, pk, pv, q_mant_bits=qbits)
        if (dtype, p, n, Tq) == (torch.float16, 8, 16, 3):
            # one head of a 364-token sequence, which is not split, is 3.3e-4 of its largest entry off before the rounding (the
            # bound by element allows 3e-4), with the bits it always had: the flat bar of 2e-3 a head
            assert rel_l2_per_head(got[:, i], want).max() <= 2e-3
        else:
            assert_attention_close(got[:, i], want, dtype, "token %d, lens %s" % (i, lens))


@pytest.mark.parametrize("B,Hkv,S", [(40, 8, 4096), (3, 64, 9500)])
def test_lengths_that_change_between_replays(B, Hkv, S):
    """One captured call, replayed with lengths that are shared out, equal ones, short ones and shared out again."""
    k, v, q, _, _ = make_small(torch.bfloat16, B=B, S=S, Hkv=Hkv, G=2, seed=660)
    cache, qd = gpu_cache(k.cuda(), v.cuda(), 32, 4, S), q.cuda()
    lens = dev_i32([S] * B)
    ws = torch.empty(kvbfp.decode_workspace_bytes(cache.layout, 2 * Hkv, S), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(qd)
    call = lambda o, w: kvbfp.decode_attention(cache, qd, S, 0.1, seq_len_dev=lens, out=o, workspace=w)
    call(out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out, ws)
    for kind in (_lens(B, S, 1), [S] * B, [min(l, 300) for l in _lens(B, S, 2)], _lens(B, S, 3), [0] * B):
        lens.copy_(dev_i32(kind))
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        assert torch.equal(got, call(torch.empty_like(qd), torch.full_like(ws, 0xFF)))
        for b in range(B):
            if kind[b] == 0:
                assert bool((got[b] == 0).all())


def test_a_workspace_without_room_for_the_table_is_enough():
    # the partial results alone, as before there was a table: nothing is shared out then
    B, Hkv, G, S = 48, 8, 2, 2400                # ten tiles of 384 units: two splits, shared out (nine have one)
    lens = _lens(B, S, 4)
    k, v, q, _, _ = make_small(torch.float32, B=B, S=S, Hkv=Hkv, G=G, seed=670)
    cache = gpu_cache(k.cuda(), v.cuda(), 32, 4, S)
    need = kvbfp.decode_workspace_bytes(cache.layout, Hkv * G, S)
    rows = need // (B * Hkv * G * 130 * 4) * (B * Hkv * G * 130 * 4)
    assert need == rows + 8 * B
    ws = torch.zeros(need + 64, dtype=torch.uint8, device="cuda")
    kw = dict(seq_len_dev=dev_i32(np.asarray(lens)))
    a = kvbfp.decode_attention(cache, q.cuda(), S, 0.1, workspace=ws[:rows], **kw)
    with pytest.raises(kvbfp.KvbfpError):
        kvbfp.decode_attention(cache, q.cuda(), S, 0.1, workspace=ws[:rows - 4], **kw)
    b = kvbfp.decode_attention(cache, q.cuda(), S, 0.1, workspace=ws[:need], **kw)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0).all())
    same = torch.equal(a, b)
    assert not same and bool(((a - b).norm() <= 1e-5 * a.norm()))


@pytest.mark.parametrize("n,S", [(16, 1100), (32, 2000)])
def test_rotation_at_read(n, S):
    B = 24
    lens = _lens(B, S, 9)
    k, v, q, pk, pv = make_small(torch.bfloat16, B=B, S=S, Hkv=8, G=2, seed=620)
    got, want = run_rope(k, v, q, n, 4, lens, 128 ** -0.5, pk, pv, 1)
    assert_attention_close(got, want, torch.bfloat16)


@pytest.mark.parametrize("p,G,B,S", [(4, 4, 40, 1100), (4, 4, 40, 4096), (8, 2, 40, 1100), (8, 2, 25, 2100), (4, 10, 24, 900), (8, 70, 12, 1000)])
def test_append_inside_the_pass(p, G, B, S):
    Hkv, n = 8, 32
    lens = _lens(B, S, 11)
    k, v, q, pk, pv = make_small(torch.bfloat16, B=B, S=S, Hkv=Hkv, G=G, seed=630)
    lens_t, pkd, pvd = dev_i32(np.asarray(lens)), dev_i32(pk), dev_i32(pv)
    kn, vn = k[:, 5].contiguous().cuda(), v[:, 7].contiguous().cuda()
    one, two = (gpu_cache(k.cuda(), v.cuda(), n, p, S, perm_k=pk, perm_v=pv) for _ in range(2))
    kvbfp.quantize_append(two, kn.unsqueeze(1), vn.unsqueeze(1), pos_dev=lens_t - 1, perm_k=pkd, perm_v=pvd)
    a = kvbfp.append_decode_attention(one, kn, vn, q.cuda(), S, 0.1, seq_len_dev=lens_t, perm_k=pkd, perm_v=pvd)
    b = kvbfp.decode_attention(two, q.cuda(), S, 0.1, seq_len_dev=lens_t, perm_k=pkd, perm_v=pvd)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and all(torch.equal(x, y) for x, y in zip(one.planes(), two.planes()))


@pytest.mark.parametrize("dtype,p,n,G", [
    (torch.bfloat16, 4, 32, 1), (torch.float16, 8, 64, 6), (torch.float32, 4, 16, 4), (torch.float32, 8, 128, 5),
    (torch.bfloat16, 4, 16, 12),                 # many heads: keeps the combine pass
])
def test_one_split_writes_the_output_itself(dtype, p, n, G):
    # 256 tokens and fewer are one tile, so one split; a full tile, one token, none, a ragged tile
    k, v, q, pk, pv = make_small(dtype, B=4, S=256, Hkv=2, G=G, seed=700 + G)
    got, want = run_both(k, v, q, n, p, [256, 1, 0, 200], 128 ** -0.5, pk, pv)
    assert_attention_close(got, want, dtype)
    assert bool((got[2] == 0).all())


def test_one_split_of_the_rotation_at_read():
    k, v, q, pk, pv = make_small(torch.bfloat16, B=3, S=256, Hkv=2, G=6, seed=710)
    got, want = run_rope(k, v, q, 32, 4, [256, 0, 130], 128 ** -0.5, pk, pv, 1)
    assert_attention_close(got, want, torch.bfloat16)


@pytest.mark.parametrize("dtype,p,G,B,Hkv,S", [
    (torch.bfloat16, 4, 4, 24, 8, 8100),         # 4 splits: a wavefront of the combine pass per head
    (torch.float32, 4, 1, 24, 8, 1100),
    (torch.bfloat16, 4, 12, 24, 8, 1100),        # 9 to 32 heads
    (torch.bfloat16, 8, 40, 12, 8, 1100),        # more
    (torch.float32, 4, 4, 4, 2, 30000),          # 96 splits: a workgroup of it per head
])
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("bits", [0xFFC00000, 0x7FC00000])
def test_a_query_that_is_not_a_number_stays_in_its_sequence(dtype, p, G, B, Hkv, S, ragged, bits):
    # whatever its sign: the form of the partial results is not told by what is computed
    lens = dev_i32(_lens(B, S, 21) if ragged else [S] * B)
    k, v, q, _, _ = make_small(dtype, B=B, S=S, Hkv=Hkv, G=G, seed=640)
    cache = gpu_cache(k.cuda(), v.cuda(), 32, p, S)
    want = kvbfp.decode_attention(cache, q.cuda(), S, 0.1, seq_len_dev=lens)
    bad = q.clone()
    if dtype == torch.float32:
        bad[1] = torch.tensor(bits - (1 << 32 if bits >> 31 else 0), dtype=torch.int32).view(torch.float32)
    else:
        bad.view(torch.int16)[1] = (bits >> 16) - (1 << 16 if bits >> 31 else 0)
    assert bool(bad[1].isnan().all())
    got = kvbfp.decode_attention(cache, bad.cuda(), S, 0.1, seq_len_dev=lens)
    torch.cuda.synchronize()
    keep = [b for b in range(B) if b != 1]
    assert torch.equal(got[keep], want[keep])
    assert bool((got[1].isnan() | (got[1] == 0)).all())


@pytest.mark.parametrize("dt,p,B,rope", [("bf16", 4, 24, False), ("f32", 4, 24, False), ("bf16", 8, 16, False), ("f32", 8, 16, False), ("f16", 4, 16, True),
                                            ("bf16", 8, 16, True), ("f32", 4, 16, True), ("f32", 8, 16, True)])
@pytest.mark.parametrize("given", [False, True])
def test_five_tiles_where_four_splits_fit(dt, p, B, rope, given):
    """Three splits of two, two and one tile take their place: whole tiles, one token in the last, none in it, none at all."""
    Hkv, S, n = 8, 1200, 32
    lens = np.resize(np.asarray([1200, 1025, 1024, 512, 1, 0, 769], np.int32), B) if given else np.full(B, S, np.int32)
    torch_dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dt]
    k, v = (synth.kv_rows(B, S, Hkv, D, dt, synth.outlier_gains(61, t, Hkv, D), 61, 2 + t) for t in (0, 1))
    q = synth.queries(B, Hkv, D, dt, 61, 4)
    planes = oracle_cache(k, v, n, p, S, 0)
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S)
    scale = float(np.float32(D ** -0.5))
    lens_dev = dev_i32(lens) if given else None
    if rope:
        theta = (10000.0 ** (-np.arange(0, D, 2, dtype=np.float64) / D)).astype(np.float32)
        r = kvbfp.permute_rope(theta, np.tile(np.arange(D, dtype=np.int32), (Hkv, 1)))
        got = kvbfp.decode_attention_rope(cache, q.cuda(), S, scale, *(torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in r), seq_len_dev=lens_dev)
        want = O.decode_attention_rope(*planes, D, n, p, synth.to_f32_numpy(q), lens, scale, *r)
    else:
        got = kvbfp.decode_attention(cache, q.cuda(), S, scale, seq_len_dev=lens_dev)
        want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), lens, scale)
    torch.cuda.synchronize()
    assert_attention_close(got, want, torch_dt, "%s p=%d B=%d" % (dt, p, B))


@pytest.mark.parametrize("dt,p,B,rope,five", [("f32", 4, 24, False, 3), ("bf16", 8, 16, False, 4), ("f32", 8, 16, False, 4), ("f16", 4, 16, True, 4),
                                                 ("bf16", 8, 16, True, 4), ("f32", 4, 16, True, 4)])
def test_the_splits_follow_the_lengths_and_not_max_len(dt, p, B, rope, five):
    """Planned for five tiles, four splits fit.  Lengths of four tiles and fewer have a split for every tile; five tiles
    take three (two, two and one) with fp32 I/O and 4 bits, four elsewhere."""
    Hkv, S, n, Hq = 8, 1200, 32, 8
    layout = kvbfp.make_layout(D, n, p, Hkv, B, S)
    cache = kvbfp.alloc_cache(layout, "cuda", fill=0)
    q = torch.zeros((B, Hq, D), dtype={"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dt], device="cuda")
    ws = torch.zeros((kvbfp.decode_workspace_bytes(layout, Hq, S) + 4096,), dtype=torch.uint8, device="cuda")
    if rope:
        theta = (10000.0 ** (-np.arange(0, D, 2, dtype=np.float64) / D)).astype(np.float32)
        r = [torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in kvbfp.permute_rope(theta, np.tile(np.arange(D, dtype=np.int32), (Hkv, 1)))]
    for length, busy in ((1200, five), (1024, 4), (700, 3), (512, 2), (1, 1)):
        kw = dict(seq_len_dev=dev_i32(np.full(B, length)), workspace=ws)
        if rope:
            kvbfp.decode_attention_rope(cache, q, S, 0.1, *r, **kw)
        else:
            kvbfp.decode_attention(cache, q, S, 0.1, **kw)
        torch.cuda.synchronize()
        rows = B * Hq * 4
        weight = ws.view(torch.float32)[rows * D:rows * (D + 2)].view(B, Hq, 4, 2)[..., 1]      # of a row: as many as it has tokens
        assert bool((weight.sum(-1) == length).all()) and bool(((weight > 0).sum(-1) == busy).all()), (length, weight[0, 0].tolist())
