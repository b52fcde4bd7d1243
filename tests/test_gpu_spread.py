"""Sequences of different lengths: the workgroups of a kv-head shared out by the lengths (decode_spans.h), for every split
pass that does so, against the oracle.  The batch and head counts leave fewer splits than tiles, which is where it applies."""
import numpy as np
import pytest
import torch

from test_gpu_attention import make_small, run_both
from test_gpu_rope_at_read import run_both as run_rope
from util import assert_attention_close, dev_i32, gpu_cache
from paper_2403_20137_amd import kvbfp

pytestmark = pytest.mark.gpu


def _lens(B, S, seed, long_only=False):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 100, B) if long_only else np.exp(rng.uniform(0, np.log(S), B)).astype(np.int64)
    lens[rng.integers(B)] = S
    if B > 3:
        lens[np.flatnonzero(lens != S)[0]] = 0
    return [int(x) for x in lens]


@pytest.mark.parametrize("dtype,p,n,G,B,Hkv,S", [
    (torch.bfloat16, 4, 32, 1, 70, 8, 1100),      # more than 64 sequences, two splits of five tiles; LDS pipeline
    (torch.float16, 8, 16, 1, 40, 8, 1100),       # 8-bit pipeline
    (torch.float32, 4, 16, 1, 40, 8, 900),        # register-staged passes
    (torch.float32, 8, 32, 1, 40, 8, 900),
    (torch.bfloat16, 4, 32, 12, 24, 8, 900),      # 9 to 32 heads, tiles of 128
    (torch.bfloat16, 4, 16, 40, 12, 8, 700),      # more heads, tiles of 64
    (torch.bfloat16, 4, 32, 4, 3, 64, 1500),      # three sequences
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
    B, S = 2, 13000                              # 2 x 8 units: 48 splits, 51 tiles; the 32-channel combine
    k, v, q, pk, pv = make_small(torch.bfloat16, B=B, S=S, Hkv=8, G=1, seed=610)
    got, want = run_both(k, v, q, 32, 4, [S, 300], 128 ** -0.5, pk, pv)
    assert_attention_close(got, want, torch.bfloat16)


@pytest.mark.parametrize("n", [16, 32])
def test_rotation_at_read(n):
    B, S = 24, 1100
    lens = _lens(B, S, 9)
    k, v, q, pk, pv = make_small(torch.bfloat16, B=B, S=S, Hkv=8, G=2, seed=620)
    got, want = run_rope(k, v, q, n, 4, lens, 128 ** -0.5, pk, pv, 1)
    assert_attention_close(got, want, torch.bfloat16)


@pytest.mark.parametrize("p,G", [(4, 4), (8, 2), (4, 10)])
def test_append_inside_the_pass(p, G):
    B, Hkv, S, n = 40, 8, 1100, 32
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
    (torch.bfloat16, 4, 4, 24, 8, 1100),         # 4 splits: a wavefront of the combine pass per head
    (torch.float32, 4, 1, 24, 8, 1100),
    (torch.bfloat16, 4, 12, 24, 8, 1100),        # 9 to 32 heads
    (torch.bfloat16, 8, 40, 12, 8, 1100),        # more
    (torch.bfloat16, 4, 4, 2, 8, 13000),         # 48 splits: a workgroup of it per head
    (torch.float32, 4, 4, 2, 8, 13000),
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
