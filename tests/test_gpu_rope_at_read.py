"""GPU parity of decode attention over keys cached before the rotary embedding and rotated at read
with the reordered parameters (Sec. III; Alg. 1 step 5), against the oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import kvbfp_oracle as O
from paper_2403_20137_amd import kvbfp, synth
from test_gpu_attention import make_small
from util import assert_attention_close, assert_planes_equal, dev_i32, gpu_cache, oracle_cache

pytestmark = pytest.mark.gpu

D = 128


def llama_theta(base=10000.0):
    return (base ** (-np.arange(D // 2, dtype=np.float64) / (D // 2))).astype(np.float32)


def run_both(k, v, q, n, p, lens, scale, pk, pv, pairs, S_max=None, theta=None, profile=False):
    B, S, Hkv, _ = k.shape
    S_max = S if S_max is None else S_max
    theta = llama_theta() if theta is None else theta
    ident = np.tile(np.arange(D, dtype=np.int32), (Hkv, 1))
    planes = oracle_cache(k, v, n, p, S_max, 0, pk, pv)
    cache = gpu_cache(k.cuda(), v.cuda(), n, p, S_max, perm_k=pk, perm_v=pv)
    assert_planes_equal(cache, planes, "cache before attention")
    th_o, pa_o, sg_o = O.permute_rope(theta, ident if pk is None else pk, pairs)
    want = O.decode_attention_rope(*planes, D, n, p, synth.to_f32_numpy(q), lens, float(np.float32(scale)),
                                   th_o, pa_o, sg_o, perm_k=pk, perm_v=pv)
    th, pa, sg = kvbfp.permute_rope(theta, ident if pk is None else pk, pairs)      # the library's own host call
    sl = dev_i32(np.broadcast_to(np.asarray(lens), (B,)))
    got = kvbfp.decode_attention_rope(cache, q.cuda(), int(np.max(lens)), float(np.float32(scale)),
                                      torch.from_numpy(th).cuda(), torch.from_numpy(pa).cuda(),
                                      torch.from_numpy(sg).cuda(), seq_len_dev=sl, perm_k=dev_i32(pk),
                                      perm_v=dev_i32(pv), profile=profile)
    torch.cuda.synchronize()
    return got, want


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("p,n", [(4, 16), (4, 32), (4, 128), (8, 16), (8, 64)])
@pytest.mark.parametrize("G,pairs", [(1, 0), (4, 1), (6, 0)])
def test_rotation_at_read_matches_oracle(dtype, p, n, G, pairs):
    # 700 tokens: two full 256-token tiles and a ragged third; the second sequence stops mid-tile
    k, v, q, pk, pv = make_small(dtype, B=2, S=700, Hkv=2, G=G, seed=120 + G)
    got, want = run_both(k, v, q, n, p, [700, 259], 128 ** -0.5, pk, pv, pairs, S_max=720)
    assert_attention_close(got, want, dtype, "p=%d n=%d G=%d pairs=%d" % (p, n, G, pairs))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rotation_is_not_a_no_op_and_rows_need_not_be_reordered(dtype):
    k, v, q, _, _ = make_small(dtype, B=1, S=300, Hkv=2, G=2, seed=130)
    got, want = run_both(k, v, q, 32, 4, [300], 0.1, None, None, 1)
    assert_attention_close(got, want, dtype)
    plain = kvbfp.decode_attention(gpu_cache(k.cuda(), v.cuda(), 32, 4, 300), q.cuda(), 300, float(np.float32(0.1)))
    torch.cuda.synchronize()
    assert (plain.double().cpu() - got.double().cpu()).norm() > 1e-2 * got.double().cpu().norm()


def test_token_indices_beyond_100k_keep_fp32_accuracy():
    # angles up to 1.3e5 radians at the highest frequency (theta = 1): 512 splits start all along the sequence (two of them step
    # their phasors to a second tile, the others have one), and fp32 I/O holds the 1e-5 bar
    S = 131072 + 300
    k, v, q, pk, pv = make_small(torch.float32, B=1, S=S, Hkv=1, G=2, seed=140)
    got, want = run_both(k, v, q, 32, 4, [S], 128 ** -0.5, pk, pv, 1)
    assert_attention_close(got, want, torch.float32)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_token_indices_beyond_100k_with_16_bit_io(dtype):
    # the matrix-core pass: per-tile phasors stepped in fp32 from a double-precision start over 45 tiles
    # per wavefront (12 splits), angles up to 1.3e5 radians
    S = 131072 + 300
    k, v, q, pk, pv = make_small(dtype, B=1, S=S, Hkv=1, G=4, seed=141)
    got, want = run_both(k, v, q, 32, 4, [S], 128 ** -0.5, pk, pv, 1)
    assert_attention_close(got, want, dtype)


@pytest.mark.parametrize("n", [16, 32, 128])
@pytest.mark.parametrize("k_shift,q_shift", [(-100, 0), (100, 0), (0, 90), (0, -90), (-60, -50)])
def test_rotation_at_read_at_the_ends_of_the_range(n, k_shift, q_shift):
    # block exponents are applied after the matrix product and the query is normalised per 32 channels:
    # keys and queries anywhere in the fp32 range, with the softmax scale that brings the logits back
    dtype = torch.bfloat16
    B, S, Hkv, G = 2, 600, 2, 4
    g = synth.outlier_gains(6, 0, Hkv, D)
    mk = lambda t, sh: (t * 2.0 ** sh).to(dtype)
    k = mk(synth.kv_rows(B, S, Hkv, D, "f32", g, 6, 2), k_shift)
    v = synth.kv_rows(B, S, Hkv, D, "bf16", g, 6, 3)
    q = mk(synth.queries(B, Hkv * G, D, "f32", 6, 4), q_shift)
    pk = O.calibrate_perm(synth.to_f32_numpy(k[0, :64]))
    scale = float(np.float32(D ** -0.5) * np.float32(2.0 ** (-(k_shift + q_shift))))
    got, want = run_both(k, v, q, n, 4, [S, 259], scale, pk, None, 0)
    assert bool(torch.isfinite(got).all())
    assert_attention_close(got, want, dtype, "n=%d shifts k %d q %d" % (n, k_shift, q_shift))


def test_blocks_of_16_with_very_different_exponents_inside_one_chunk():
    # every second block of 16 channels 2^30 below its neighbour: the smaller block is scaled down inside
    # the conversion, and what falls below 2^-24 of the larger block's unit is dropped
    dtype = torch.bfloat16
    k, v, q, pk, pv = make_small(dtype, B=1, S=400, Hkv=2, G=4, seed=151)
    damp = torch.ones(D)
    damp[torch.arange(D) % 32 >= 16] = 2.0 ** -30
    k = (k.float() * damp).to(dtype)
    got, want = run_both(k, v, q, 16, 4, [400], 0.3, None, pv, 1)
    assert_attention_close(got, want, dtype)


def test_profile_variant_returns_the_same_result_and_two_durations():
    k, v, q, pk, pv = make_small(torch.bfloat16, B=2, S=600, Hkv=2, G=4, seed=150)
    (got, split_ms, combine_ms), want = run_both(k, v, q, 16, 4, [600, 1], 0.09, pk, pv, 0, profile=True)
    assert_attention_close(got, want, torch.bfloat16)
    assert split_ms > 0 and combine_ms > 0


@pytest.mark.parametrize("dtype,p,n", [(torch.float16, 4, 32), (torch.bfloat16, 4, 16), (torch.float32, 4, 64), (torch.float16, 8, 32)])
def test_angles_up_to_the_limit(dtype, p, n):
    # frequencies of 2^43 to 2^44 radians a token over 60 tokens: pi / 2 in one part (53 bits) is 2^-53 of 2^49, several hundredths, off
    theta = (2.0 ** np.random.default_rng(3).uniform(43, 44, D // 2)).astype(np.float32)
    k, v, q, pk, pv = make_small(dtype, B=1, S=60, Hkv=2, G=3, seed=155)
    got, want = run_both(k, v, q, n, p, [60], 0.05, pk, pv, 1, theta=theta)
    assert_attention_close(got, want, dtype, "p=%d n=%d" % (p, n))


# ---- the pass in fp32 (8-bit mantissas, fp32 I/O, exponent planes of any alignment)

@pytest.mark.parametrize("dtype,p,n", [(torch.float32, 4, 16), (torch.float32, 4, 64), (torch.float32, 8, 32), (torch.float32, 8, 128), (torch.bfloat16, 8, 16), (torch.float16, 8, 32)])
@pytest.mark.parametrize("lens,G", [([1, 63], 4), ([64, 65], 1), ([255, 257], 5), ([512, 0], 3), ([1025, 960], 2)])
def test_fp32_pass_at_the_edges_of_its_tiles(dtype, p, n, lens, G):
    # 64 tokens to a wavefront, 256 to a workgroup; one to five heads (four to a launch); an empty sequence
    k, v, q, pk, pv = make_small(dtype, B=2, S=max(lens), Hkv=2, G=G, seed=160 + G)
    got, want = run_both(k, v, q, n, p, lens, 0.13, pk, pv, G & 1, S_max=max(lens) + 3)
    assert_attention_close(got, want, dtype, "p=%d n=%d lengths %s" % (p, n, lens))


@pytest.mark.parametrize("dtype,p,n", [(torch.float32, 4, 32), (torch.float32, 8, 16), (torch.bfloat16, 8, 64)])
@pytest.mark.parametrize("k_shift,q_shift,v_shift", [(-100, 0, 0), (100, 0, 0), (0, 90, 0), (0, -90, 0), (-60, -50, 0), (0, 0, -120), (0, 0, -126), (0, 0, 110)])
def test_fp32_pass_at_the_ends_of_the_range(dtype, p, n, k_shift, q_shift, v_shift):
    # queries beyond 2^60 are normalised; value blocks with exponent bytes 1 and 2 (v 2^-126) take fp32 multiply-adds
    B, S, Hkv, G = 2, 300, 2, 4
    g = synth.outlier_gains(7, 0, Hkv, D)
    mk = lambda t, sh: (t * 2.0 ** sh).to(dtype)
    k = mk(synth.kv_rows(B, S, Hkv, D, "f32", g, 7, 2), k_shift)
    v = mk(synth.kv_rows(B, S, Hkv, D, "f32", g, 7, 3), v_shift)
    q = mk(synth.queries(B, Hkv * G, D, "f32", 7, 4), q_shift)
    scale = float(np.float32(D ** -0.5) * np.float32(2.0 ** (-(k_shift + q_shift))))
    got, want = run_both(k, v, q, n, p, [S, 131], scale, None, None, 1)
    assert bool(torch.isfinite(got).all())
    if v_shift == -126 and dtype == torch.float32:      # subnormal outputs: the step of fp32 there on top of the bar
        err = np.abs(got.double().cpu().numpy() - want)
        assert np.all(err <= 2.0 ** -149 + 1e-5 * np.abs(want).max(axis=-1, keepdims=True))
    else:
        assert_attention_close(got, want, dtype, "p=%d n=%d shifts k %d q %d v %d" % (p, n, k_shift, q_shift, v_shift))


@pytest.mark.parametrize("n", [16, 128])
def test_fp32_pass_takes_the_largest_exponent_bytes(n):
    # three tokens with values of 2^125 (8 bits: bytes 252 and up do not fit the conversion to bf16)
    g = torch.Generator().manual_seed(9)
    k, q = torch.randn(1, 3, 2, D, generator=g), torch.randn(1, 8, D, generator=g)
    v = (torch.rand(1, 3, 2, D, generator=g) - 0.5) * 2.0 ** 125
    v[..., ::16] = 2.0 ** 125.5
    got, want = run_both(k, v, q, n, 8, [3], 0.2, None, None, 0)
    assert_attention_close(got, want, torch.float32)


@pytest.mark.parametrize("dtype,p,n", [(torch.bfloat16, 4, 16), (torch.bfloat16, 4, 32), (torch.float32, 8, 64), (torch.float32, 4, 128)])
def test_rotation_over_exponent_planes_of_any_alignment(dtype, p, n):
    k, v, q, pk, pv = make_small(dtype, B=2, S=300, Hkv=2, G=4, seed=170)
    planes = oracle_cache(k, v, n, p, 300, 0, pk, pv)
    whole = gpu_cache(k.cuda(), v.cuda(), n, p, 300, perm_k=pk, perm_v=pv)
    moved = []
    for e in (whole.k_exp, whole.v_exp):
        room = torch.zeros(e.numel() + 16, dtype=torch.uint8, device="cuda")
        room[1:1 + e.numel()] = e.reshape(-1)
        moved.append(room[1:1 + e.numel()].reshape(e.shape))
        assert moved[-1].data_ptr() % 16 == 1
    cache = kvbfp.Cache(whole.layout, whole.k_mant, moved[0], whole.v_mant, moved[1])
    r = O.permute_rope(llama_theta(), pk, 0)
    want = O.decode_attention_rope(*planes, D, n, p, synth.to_f32_numpy(q), [300, 70], 0.1, *r, perm_k=pk, perm_v=pv)
    got = kvbfp.decode_attention_rope(cache, q.cuda(), 300, float(np.float32(0.1)), *(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in r),
                                      seq_len_dev=dev_i32([300, 70]), perm_k=dev_i32(pk), perm_v=dev_i32(pv))
    torch.cuda.synchronize()
    assert_attention_close(got, want, dtype, "p=%d n=%d" % (p, n))


@pytest.mark.parametrize("dtype,p,n,G,lens,Hkv", [(torch.float32, 4, 32, 9, [700, 259], 2), (torch.bfloat16, 8, 16, 16, [300, 0], 3), (torch.float16, 4, 64, 35, [513, 64], 2)])
def test_all_heads_of_a_call_in_one_launch(dtype, p, n, G, lens, Hkv):
    # groups of four heads with a last one of fewer; more than 32 heads take the fp32 pass with 4 bits and 16-bit I/O too
    k, v, q, pk, pv = make_small(dtype, B=2, S=max(lens), Hkv=Hkv, G=G, seed=180 + G)
    got, want = run_both(k, v, q, n, p, lens, 0.11, pk, pv, 1)
    assert_attention_close(got, want, dtype, "p=%d n=%d G=%d" % (p, n, G))


def test_a_call_of_many_heads_over_short_sequences_costs_little_more_than_one_of_four():
    # 16 heads are 32 workgroups in place of 8: launched one group after the other a call took 3.3 times as long
    S, times = 300, {}
    for G in (4, 16):
        k, v, q, pk, pv = make_small(torch.bfloat16, B=1, S=S, Hkv=8, G=G, seed=190)
        cache = gpu_cache(k.cuda(), v.cuda(), 32, 8, S, perm_k=pk, perm_v=pv)
        r = [torch.from_numpy(x).cuda() for x in kvbfp.permute_rope(llama_theta(), pk, 1)]
        qd, out = q.cuda(), torch.empty_like(q, device="cuda")
        ws = torch.empty(kvbfp.decode_workspace_bytes(cache.layout, 8 * G, S), dtype=torch.uint8, device="cuda")
        call = lambda: kvbfp.decode_attention_rope(cache, qd, S, 0.1, *r, perm_k=dpk, perm_v=dpv, out=out, workspace=ws)
        dpk, dpv = dev_i32(pk), dev_i32(pv)
        call()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(50):
                call()
        graph.replay()
        got = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            got.append(a.elapsed_time(b))
        times[G] = min(got)
    assert times[16] < 2 * times[4], times


def _unit(cache, q, b, h, G, n, p, length, scale, r, pk, pv):
    """The oracle's output of one (sequence, kv-head) from the cache's bytes (compared with the oracle's own cast elsewhere)."""
    planes = [x[b:b + 1, h:h + 1].cpu().numpy() for x in cache.planes()]
    one = [None if x is None else np.ascontiguousarray(x[h:h + 1]) for x in (*r, pk, pv)]
    return O.decode_attention_rope(*planes, D, n, p, synth.to_f32_numpy(q[b:b + 1, h * G:(h + 1) * G].cpu()), [length], scale, *one[:3], perm_k=one[3], perm_v=one[4])


@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("light", [112, 124, 131, 141])
@pytest.mark.parametrize("tiles", [1, 3])
def test_light_weights_beside_a_heavy_one_keep_their_bits(p, light, tiles):
    # one token 2^light as heavy as every other one, whose values are 2^120 times as large; three tiles: 512 units have one split, the heavy token is
    # in the second tile of a wavefront and what the first one left is scaled by 2^-light.  Frequencies are 0, the second head sees no heavy token.
    B, Hkv, S, at, n, G = (1, 1, 200, 70, 32, 2) if tiles == 1 else (64, 8, 600, 256 + 70, 16, 2)
    gen = torch.Generator(device="cuda").manual_seed(light)
    k = torch.zeros(B, S, Hkv, D, device="cuda")
    k[:, at, :, 0] = 1.0
    v = torch.randn(B, S, Hkv, D, generator=gen, device="cuda") * 2.0 ** 100
    v[:, at] *= 2.0 ** -120
    q = torch.zeros(B, Hkv * G, D, device="cuda")
    q[:, ::G, 0] = 1.0
    scale = float(np.float32(light * np.log(2.0)))
    cache = gpu_cache(k, v, n, p, S)
    ident = np.tile(np.arange(D, dtype=np.int32), (Hkv, 1))
    r = kvbfp.permute_rope(np.zeros(D // 2, np.float32), ident, 0)
    got = kvbfp.decode_attention_rope(cache, q, S, scale, *(torch.from_numpy(x).cuda() for x in r))
    torch.cuda.synchronize()
    for b, h in {(0, 0), (B // 2, Hkv // 2), (B - 1, Hkv - 1)}:
        want = _unit(cache, q, b, h, G, n, p, S, scale, r, None, None)[0]
        top = float(v[b, :, h].abs().max())
        # the bar of fp32, on the light part what rounding a score of `light` twice does to its power, and fp32's step below 2^-126: half of 2^-149 a token
        # and for the scaling of a tile's sum
        bar = [1e-5 + 2 * light * np.log(2.0) * 2.0 ** -23, 1e-5]
        step = [2.0 ** -149 * top * S, 0.0]
        for g in range(G):
            err = np.linalg.norm(got[b, h * G + g].double().cpu().numpy() - want[g])
            assert err <= bar[g] * np.linalg.norm(want[g]) + step[g], (b, h, g, err, np.linalg.norm(want[g]))


@pytest.mark.parametrize("dtype,p,n,G", [(torch.bfloat16, 8, 16, 4), (torch.float16, 8, 64, 1), (torch.bfloat16, 8, 128, 6), (torch.float32, 8, 32, 3), (torch.float32, 8, 16, 5),
                                         (torch.float32, 4, 32, 4), (torch.float32, 4, 128, 2), (torch.float16, 4, 64, 33)])
@pytest.mark.parametrize("B,S,ragged", [(16, 2700, False), (17, 700, False), (24, 2000, True)])
def test_fp32_pass_over_several_tiles_of_a_wavefront(dtype, p, n, G, B, S, ragged):
    # 128 or 192 units (times the groups of four heads): 4 splits or fewer, three tiles and more each, the last one ragged; the phasor steps, the keys
    # requested ahead are used, the sums are scaled.  17 x 8 units of two groups: three splits of a tile, in two rounds.  Lengths that differ: the
    # workgroups are shared out.
    Hkv = 8 if G <= 8 else 2
    name = {torch.float32: "f32", torch.float16: "f16", torch.bfloat16: "bf16"}[dtype]
    gains = synth.outlier_gains(11, 0, Hkv, D)
    k, v = (synth.kv_rows(B, S, Hkv, D, name, gains, 11, 2 + t, "cuda") for t in (0, 1))
    q = synth.queries(B, Hkv * G, D, name, 11, 4, "cuda")
    pk = O.calibrate_perm(synth.to_f32_numpy(k[0, :64].cpu()))
    lens = [S] * B
    if ragged:
        rng = np.random.default_rng(B + G)
        lens = [int(x) for x in np.exp(rng.uniform(np.log(20), np.log(S), B))]
        lens[3], lens[B - 1], lens[B // 2] = S, 0, 1025
    cache = gpu_cache(k, v, n, p, S, perm_k=pk, perm_v=pk)
    r = kvbfp.permute_rope(llama_theta(500000.0), pk, 1)
    scale = float(np.float32(D ** -0.5))
    got = kvbfp.decode_attention_rope(cache, q, S, scale, *(torch.from_numpy(x).cuda() for x in r), seq_len_dev=dev_i32(np.asarray(lens)) if ragged else None,
                                      perm_k=dev_i32(pk), perm_v=dev_i32(pk))
    torch.cuda.synchronize()
    for b, h in [(0, 0), (1, Hkv - 1), (3, Hkv - 1), (B // 2, 1), (B - 1, 0)]:
        want = _unit(cache, q, b, h, G, n, p, lens[b], scale, r, pk, pk)
        assert_attention_close(got[b:b + 1, h * G:(h + 1) * G], want, dtype, "p=%d n=%d G=%d (%d, %d) of %d" % (p, n, G, b, h, lens[b]))


@pytest.mark.parametrize("dtype,p,n", [(torch.float32, 4, 16), (torch.float32, 8, 128), (torch.bfloat16, 8, 32)])
def test_heads_of_very_different_ranges_beside_each_other(dtype, p, n):
    # above 2^60 (a softmax of one token), zero (the mean), ordinary and below 2^-60 in one group of four: all are normalised together
    k, v, q, pk, pv = make_small(dtype, B=2, S=300, Hkv=2, G=5, seed=195)
    q = (q.float().view(2, 2, 5, D) * torch.tensor([2.0 ** 70, 0.0, 1.0, 2.0 ** -70, 1.0]).view(1, 1, 5, 1)).to(dtype).view(2, 10, D)
    got, want = run_both(k, v, q, n, p, [300, 67], 0.11, pk, pv, 1)
    assert bool(torch.isfinite(got).all())
    assert_attention_close(got, want, dtype, "p=%d n=%d" % (p, n))
