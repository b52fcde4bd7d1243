"""Short sequences whose tokens all go to one workgroup of eight wavefronts and whose output is written without a combine pass
(16-bit I/O, up to 8 heads per kv-head), against the oracle: at the edges of its 64-token and 512-token tiles, for lengths that
differ, with the current token appended, over pages, with several query tokens and with the integer score product."""
import numpy as np
import pytest
import torch

from oracle import kvbfp_oracle as O
from paper_2403_20137_amd import kvbfp, synth
from test_gpu_append_decode import _case
from test_gpu_attention import make_small, run_both
from test_gpu_paged import fill_both
from util import assert_attention_close, dev_i32

pytestmark = pytest.mark.gpu
D = 128


# the longest sequence decides: 257 tokens and up (fewer are one split of four wavefronts), 512 are one tile of the workgroup; the last
# lengths are on either side of the lines for these few units (test_where_the_lines_lie)
@pytest.mark.parametrize("p,n,G,longest", [(4, 32, 4, 1024), (4, 16, 1, 1025), (4, 128, 8, 768), (4, 64, 5, 769), (8, 16, 2, 768), (8, 32, 4, 769), (8, 64, 8, 512), (8, 128, 7, 513)])
def test_current_token_at_the_edges_of_the_tiles(p, n, G, longest):
    dtype = torch.float16 if n == 64 else torch.bfloat16
    for i, lens in enumerate([[257, 64, 0, 1], [512, 449, 65, 448], [513, 512, 128, 256], [longest, 577, 513, 511]]):
        lens = [min(l, longest) for l in lens]
        _case(dtype, n, p, G, lens, max(lens) + 5, i & 1, seed=400 + n + G + i)


@pytest.mark.parametrize("p,n,G,page", [(4, 32, 4, 16), (4, 32, 8, 64), (8, 16, 4, 32), (8, 64, 6, 256), (4, 128, 2, 128)])
@pytest.mark.parametrize("lens", [[512, 500, 17], [513, 64, 300], [300, 512, 65]])
def test_over_pages(p, n, G, page, lens):
    S = max(lens)
    k, v, q, pk, pv = make_small(torch.bfloat16, B=3, S=S, Hkv=2, G=G, seed=410 + G)
    pool, table, planes = fill_both(k, v, n, p, page, -(-S // page) + 1, lens, pk, pv, seed=G + page)
    scale = float(np.float32(128 ** -0.5))
    for qbits in (0, 8):
        want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q), lens, scale, pk, pv, q_mant_bits=qbits)
        got = kvbfp.decode_attention_paged(pool, table, q.cuda(), S, scale, q_mant_bits=qbits, seq_len_dev=dev_i32(lens),
                                           perm_k=dev_i32(pk), perm_v=dev_i32(pv))
        torch.cuda.synchronize()
        assert_attention_close(got, want, torch.bfloat16, "p=%d n=%d G=%d page=%d lengths %s q bits %d" % (p, n, G, page, lens, qbits))


@pytest.mark.parametrize("p,n,G,Tq", [(4, 32, 2, 2), (4, 16, 1, 8), (8, 32, 2, 3)])
def test_several_query_tokens(p, n, G, Tq):
    # the last tokens of a tile are hidden from some heads only
    lens = [515, 512, 2, 449]
    k, v, _, pk, pv = make_small(torch.bfloat16, B=4, S=515, Hkv=2, G=G, seed=420)
    q = torch.stack([synth.queries(4, 2 * G, D, "bf16", 421 + i, 4) for i in range(Tq)], dim=1)
    cache = kvbfp.alloc_cache(kvbfp.make_layout(D, n, p, 2, 4, 515), "cuda", fill=0)
    kvbfp.quantize_append(cache, k.cuda(), v.cuda(), perm_k=dev_i32(pk), perm_v=dev_i32(pv))
    planes = [x.cpu().numpy() for x in cache.planes()]
    got = kvbfp.decode_attention_multi(cache, q.cuda(), 515, 0.1, seq_len_dev=dev_i32(lens), perm_k=dev_i32(pk), perm_v=dev_i32(pv))
    torch.cuda.synchronize()
    for i in range(Tq):
        seen = [max(l - (Tq - 1 - i), 0) for l in lens]
        want = O.decode_attention(*planes, D, n, p, synth.to_f32_numpy(q[:, i]), seen, float(np.float32(0.1)), pk, pv)
        assert_attention_close(got[:, i], want, torch.bfloat16, "query token %d of %d" % (i, Tq))


@pytest.mark.parametrize("p,n,G,S", [(4, 32, 4, 1600), (4, 32, 4, 1500), (8, 32, 4, 900), (8, 32, 4, 768), (8, 16, 4, 700), (4, 16, 8, 1280)])
def test_many_units_take_it_for_longer_sequences(p, n, G, S):
    # 128 units (4 sequences x 32 kv-heads): the line between one workgroup and splits lies higher; checked on both sides of it.  (8 bits with 5 and 6
    # heads: one head of 768 is 1.1e-3 of its largest entry off with any number of splits: its logits are large, and that pass has 16 bits of the query.)
    k, v, q, pk, pv = make_small(torch.bfloat16, B=4, S=S, Hkv=32, G=G, seed=430)
    got, want = run_both(k, v, q, n, p, [S, 513, 1, S - 64], 0.1, pk, pv)
    assert_attention_close(got, want, torch.bfloat16, "p=%d n=%d G=%d S=%d" % (p, n, G, S))


@pytest.mark.parametrize("p,n,G,longest,qbits", [(8, 16, 4, 768, 0), (8, 32, 4, 700, 8), (8, 64, 7, 640, 8), (8, 128, 8, 577, 0), (4, 32, 4, 1500, 0), (4, 16, 8, 1280, 8)])
def test_current_token_in_a_later_tile_with_many_units(p, n, G, longest, qbits):
    # 128 units: one workgroup beyond one tile of 512 tokens for 8 bits too
    _case(torch.bfloat16, n, p, G, [longest, 513, 577, 64], longest, True, seed=440 + n, qbits=qbits, Hkv=32, units=[(0, 0), (0, 31), (1, 7), (2, 19), (3, 30)])


@pytest.mark.parametrize("B,p,G,page,qbits,longest", [
    (1, 4, 4, 0, 0, 1024), (1, 4, 4, 0, 8, 1024), (1, 4, 4, 64, 0, 1024), (1, 4, 8, 0, 0, 768), (1, 4, 8, 16, 0, 768), (1, 8, 1, 0, 0, 512),
    (1, 8, 4, 0, 8, 512), (1, 8, 2, 256, 0, 512), (1, 8, 8, 0, 0, 512), (10, 8, 4, 0, 0, 512), (11, 8, 4, 0, 0, 768), (16, 8, 4, 0, 0, 768), (17, 8, 4, 0, 0, 952), (16, 8, 8, 64, 8, 768), (17, 8, 8, 64, 8, 952), (16, 4, 4, 64, 8, 1536), (16, 4, 5, 0, 0, 1280)])
def test_where_the_lines_lie(B, p, G, page, qbits, longest):
    # 8 units a sequence; one workgroup leaves no partial results in the workspace, splits do
    for S in (longest, longest + 1):
        q = torch.ones((B, 8 * G, D), dtype=torch.bfloat16, device="cuda")
        if page:
            pages = -(-S // page)
            cache = kvbfp.alloc_cache(kvbfp.make_layout(D, 32, p, 8, B * pages, page), "cuda", fill=0)
            table = dev_i32(np.arange(B * pages).reshape(B, pages))
            ws = torch.zeros(kvbfp.decode_workspace_bytes_paged(cache.layout, pages, B, 8 * G, S) + 256, dtype=torch.uint8, device="cuda")
            kvbfp.decode_attention_paged(cache, table, q, S, 0.1, q_mant_bits=qbits, workspace=ws)
        else:
            cache = kvbfp.alloc_cache(kvbfp.make_layout(D, 32, p, 8, B, S), "cuda", fill=0)
            ws = torch.zeros(kvbfp.decode_workspace_bytes(cache.layout, 8 * G, S) + 256, dtype=torch.uint8, device="cuda")
            if qbits:
                kvbfp.decode_attention_qbfp(cache, q, S, 0.1, qbits, workspace=ws)
            else:
                kvbfp.decode_attention(cache, q, S, 0.1, workspace=ws)
        torch.cuda.synchronize()
        assert bool(ws.any()) == (S > longest), S
