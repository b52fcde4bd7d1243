"""kvbfp_append_decode_attention, the call the benchmark times, against the oracle: the appended rows' bytes
bit for bit (Sec. II-B, Eq. (1)), the whole cache up to every sequence's length bit for bit, the output
within the attention bar (Sec. III).  On top: same cache bytes and same output bits as
kvbfp_quantize_append of the current token + kvbfp_decode_attention, whether the cast happens inside the
split pass or ahead of it."""
import numpy as np
import pytest
import torch

from oracle import kvbfp_oracle as O
from paper_2403_20137_amd import kvbfp, synth
from util import assert_attention_close, dev_i32

pytestmark = pytest.mark.gpu
D = 128
DT = {torch.float32: "f32", torch.float16: "f16", torch.bfloat16: "bf16"}


def _oracle_units(cache, got, k, v, q, lens, n, p, G, S_max, pk, pv, scale, qbits, dtype, units):
    """Recomputes the (batch, kv-head) units `units` with the oracle from the same inputs: the cast of
    rows [0, len) (the last one is the appended token) and attention over them."""
    for (b, h) in units:
        L = lens[b]
        out_unit = got[b:b + 1, h * G:(h + 1) * G]
        if L == 0:
            assert bool((out_unit == 0).all()), ("empty sequence must yield zeros", b, h)
            continue
        kk = synth.to_f32_numpy(k[b:b + 1, :L, h:h + 1])
        vv = synth.to_f32_numpy(v[b:b + 1, :L, h:h + 1])
        pkh = None if pk is None else pk[h:h + 1].cpu().numpy()
        pvh = None if pv is None else pv[h:h + 1].cpu().numpy()
        km, ke = O.quantize_append(kk, n, p, L, 0, perm=pkh)
        vm, ve = O.quantize_append(vv, n, p, L, 0, perm=pvh)
        for plane, ref, nm in ((cache.k_mant, km, "k_mant"), (cache.k_exp, ke, "k_exp"),
                               (cache.v_mant, vm, "v_mant"), (cache.v_exp, ve, "v_exp")):
            gotp = plane[b, h, :L].cpu().numpy()
            assert np.array_equal(gotp[L - 1], ref[0, 0, L - 1]), ("appended row differs from the oracle", nm, b, h)
            assert np.array_equal(gotp, ref[0, 0]), ("cache differs from the oracle", nm, b, h)
        want = O.decode_attention(km, ke, vm, ve, D, n, p, synth.to_f32_numpy(q[b:b + 1, h * G:(h + 1) * G]), [L], scale,
                                  pkh, pvh, q_mant_bits=qbits)
        assert_attention_close(out_unit, want, dtype, "append_decode_attention unit (%d,%d) n=%d p=%d" % (b, h, n, p))


def _case(dtype, n, p, G, lens, S_max, use_perm, seed, qbits=0, Hkv=2, units=None, max_len=None):
    B = len(lens)
    max_len = max(lens) if max_len is None else max_len
    S = max(max(lens), 1)
    gains = synth.outlier_gains(seed, 0, Hkv, D)
    k = synth.kv_rows(B, S, Hkv, D, DT[dtype], gains, seed, 2, "cuda")
    v = synth.kv_rows(B, S, Hkv, D, DT[dtype], gains, seed, 3, "cuda")
    q = synth.queries(B, Hkv * G, D, DT[dtype], seed, 4, "cuda")
    pk = pv = None
    if use_perm:
        g = torch.Generator().manual_seed(seed)
        pk = torch.stack([torch.randperm(D, generator=g) for _ in range(Hkv)]).to(torch.int32).cuda()
        pv = torch.stack([torch.randperm(D, generator=g) for _ in range(Hkv)]).to(torch.int32).cuda()
    layout = kvbfp.make_layout(D, n, p, Hkv, B, S_max)
    lens_t = dev_i32(np.asarray(lens))
    # the current token of sequence b is row lens[b] - 1 of k / v
    idx = torch.tensor([max(l - 1, 0) for l in lens], device="cuda")
    k_new = k[torch.arange(B, device="cuda"), idx].contiguous()      # [B][Hkv][D]
    v_new = v[torch.arange(B, device="cuda"), idx].contiguous()
    caches = []
    for _ in range(2):
        c = kvbfp.alloc_cache(layout, "cuda", fill=0xAB)
        kvbfp.quantize_append(c, k, v, perm_k=pk, perm_v=pv)             # history (the current token's slot too,
        caches.append(c)                                                  # overwritten below by both variants)
        for plane in (c.k_mant, c.k_exp, c.v_mant, c.v_exp):             # make the slot differ from the result
            for b, l in enumerate(lens):
                if l > 0:
                    plane[b, :, l - 1] = 0x5A
    a, f = caches
    scale = 0.1
    kvbfp.quantize_append(a, k_new.unsqueeze(1), v_new.unsqueeze(1), pos_dev=lens_t - 1, perm_k=pk, perm_v=pv)
    if qbits:
        want = kvbfp.decode_attention_qbfp(a, q, max_len, scale, qbits, seq_len_dev=lens_t, perm_k=pk, perm_v=pv)
    else:
        want = kvbfp.decode_attention(a, q, max_len, scale, seq_len_dev=lens_t, perm_k=pk, perm_v=pv)
    got = kvbfp.append_decode_attention(f, k_new, v_new, q, max_len, scale, seq_len_dev=lens_t, perm_k=pk, perm_v=pv,
                                        q_mant_bits=qbits)
    torch.cuda.synchronize()
    for name in ("k_mant", "k_exp", "v_mant", "v_exp"):
        assert torch.equal(getattr(a, name), getattr(f, name)), name
    assert torch.equal(got, want)
    # ... and the one-call result against the oracle (all units of a small case, sampled ones of a large one)
    if units is None:
        units = [(b, h) for b in range(B) for h in range(Hkv)]
    _oracle_units(f, got, k, v, q, lens, n, p, G, S_max, pk, pv, scale, qbits, dtype, units)


@pytest.mark.parametrize("n", [16, 32])
@pytest.mark.parametrize("G", [1, 4, 8])
@pytest.mark.parametrize("use_perm", [False, True])
def test_small_caches_equal_two_calls(n, G, use_perm):
    # lengths: full tiles + 1, mid-tile, a single token, an empty sequence
    _case(torch.bfloat16, n, 4, G, [1025, 700, 1, 0], 1100, use_perm, seed=30 + n + G)


@pytest.mark.parametrize("n,G,use_perm,qbits", [(n, *rest) for n in (16, 32) for rest in
                                                 [(1, False, 0), (2, True, 0), (2, True, 8), (12, True, 0)]] +
                         [(64, 4, True, 0), (64, 6, False, 8), (128, 1, True, 0), (128, 8, True, 0)])
def test_cast_inside_the_split_pass_equals_two_calls(n, G, use_perm, qbits):
    # In the LDS pipeline the wavefront whose 64-token tiles hold the last token casts and stores the new
    # rows itself.  4 x 64 = 256 (batch, kv-head) units ask for 3 splits (2 with 12 heads per kv-head),
    # tiles are dealt round-robin; the current tokens fall into the last tile of a sequence of seven
    # full tiles (fourth wavefront), into tile 2 (third wavefront) and into tile 5 (first wavefront),
    # and one sequence is empty.  (max_len is what the lengths may become: up to 12 x 256 tokens a sequence has one workgroup of eight.)
    _case(torch.bfloat16, n, 4, G, [1792, 700, 1300, 0], 3200, use_perm, seed=60 + n + G, qbits=qbits, Hkv=64,
          units=[(0, 0), (0, 63), (1, 17), (2, 40), (3, 5)], max_len=3200)


@pytest.mark.parametrize("n,G,use_perm,qbits", [(16, 1, True, 0), (16, 8, False, 0), (32, 4, True, 8), (64, 2, True, 0), (128, 6, True, 0)])
def test_cast_inside_the_split_pass_8_bit_mantissas(n, G, use_perm, qbits):
    # the same with 8-bit mantissas (two workgroups per compute unit: 64 x 4 units ask for 2 splits, from 7 x 256 tokens on)
    _case(torch.bfloat16, n, 8, G, [1792, 700, 1300, 0], 2000, use_perm, seed=80 + n + G, qbits=qbits, Hkv=64,
          units=[(0, 0), (0, 63), (1, 17), (2, 40), (3, 5)], max_len=2000)


def test_cast_inside_the_split_pass_fp16():
    _case(torch.float16, 32, 4, 1, [1700, 1792, 1537, 1], 3200, True, seed=77, Hkv=64,
          units=[(0, 3), (1, 63), (2, 31), (3, 0), (3, 62)], max_len=3200)


@pytest.mark.parametrize("dtype,n,p", [(torch.bfloat16, 16, 8), (torch.bfloat16, 64, 4), (torch.float32, 32, 4),
                                       (torch.float16, 128, 8)])
def test_append_ahead_of_the_split_pass_equals_two_calls(dtype, n, p):
    _case(dtype, n, p, 2, [600, 259, 0], 640, True, seed=50 + n + p)


def test_without_sequence_lengths_the_token_goes_to_the_last_position():
    B, Hkv, G, S = 2, 2, 4, 515
    gains = synth.outlier_gains(3, 0, Hkv, D)
    k = synth.kv_rows(B, S, Hkv, D, "bf16", gains, 3, 2, "cuda")
    v = synth.kv_rows(B, S, Hkv, D, "bf16", gains, 3, 3, "cuda")
    q = synth.queries(B, Hkv * G, D, "bf16", 3, 4, "cuda")
    layout = kvbfp.make_layout(D, 32, 4, Hkv, B, S)
    a, f = kvbfp.alloc_cache(layout, "cuda", fill=0), kvbfp.alloc_cache(layout, "cuda", fill=0)
    kvbfp.quantize_append(a, k, v)
    kvbfp.quantize_append(f, k[:, :-1], v[:, :-1])
    want = kvbfp.decode_attention(a, q, S, 0.1)
    got = kvbfp.append_decode_attention(f, k[:, -1:], v[:, -1:], q, S, 0.1)
    torch.cuda.synchronize()
    assert torch.equal(a.k_mant, f.k_mant) and torch.equal(a.v_exp, f.v_exp) and torch.equal(got, want)


def test_headline_configuration_in_the_launch_shape_of_the_benchmark():
    # 8 sequences x 8 kv-heads x 32769 tokens, 4 query heads per kv-head, block 32: 12 splits of 11 tiles,
    # the last one 8 tiles long -> the cast runs inside the split pass
    _case(torch.bfloat16, 32, 4, 4, [32769, 32769, 32700, 32769, 30000, 32769, 32769, 28161], 32769, True, seed=99, Hkv=8,
          units=[(0, 0), (2, 5), (4, 7), (7, 3)])
