"""The pass for fp32 I/O and 4-bit mantissas against the oracle where its tiles change: a wavefront's first, steady and last 64-token
tile, and the numbers of (batch, kv-head) units and tiles at which two or three workgroups per compute unit are planned."""
import numpy as np
import pytest
import torch

from paper_2403_20137_amd import kvbfp, synth
from test_gpu_attention import make_small, run_both
from test_gpu_append_decode import _oracle_units
from util import assert_attention_close, dev_i32

pytestmark = pytest.mark.gpu
D = 128


@pytest.mark.parametrize("n,G", [(16, 4), (32, 1), (64, 3), (128, 2), (32, 7)])
@pytest.mark.parametrize("S", [64, 255, 257, 513, 4160])
def test_edges_of_a_wavefronts_tiles(n, G, S):
    # one split of up to a tile for every wavefront, two splits, and 16 units that share a longer sequence out
    k, v, q, pk, pv = make_small(torch.float32, B=4, S=S, Hkv=4, G=G, seed=500 + n)
    got, want = run_both(k, v, q, n, 4, [S, max(S - 63, 1), (S + 1) // 2, min(65, S)], 0.1, pk, pv)
    assert_attention_close(got, want, torch.float32, "n=%d G=%d S=%d" % (n, G, S))


# 128 units: up to 4 tiles of 256 tokens have a workgroup each at two per compute unit, 5 to 7 are shared by 4 splits; 520, 640 and 704: one
# split, three per compute unit up to 512 and 768 tokens; 768 and 776: all that fit as three, and one sequence more
@pytest.mark.parametrize("n", [16, 32, 64, 128])
@pytest.mark.parametrize("B,S,lengths", [(16, 1024, False), (16, 1025, True), (16, 1536, False), (16, 1537, True), (65, 256, True), (65, 1030, True),
                                         (80, 700, True), (88, 1280, True), (88, 1281, True), (96, 1200, True), (96, 600, False), (97, 600, True)])
def test_two_and_three_workgroups_per_compute_unit(n, B, S, lengths):
    Hkv, G = 8, 4
    gains = synth.outlier_gains(n, 0, Hkv, D)
    k = synth.kv_rows(B, S, Hkv, D, "f32", gains, 510, 2, "cuda")
    v = synth.kv_rows(B, S, Hkv, D, "f32", gains, 510, 3, "cuda")
    q = synth.queries(B, Hkv * G, D, "f32", 510, 4, "cuda")
    cache = kvbfp.alloc_cache(kvbfp.make_layout(D, n, 4, Hkv, B, S), "cuda", fill=0xAB)
    kvbfp.quantize_append(cache, k, v)
    lens = [S - (37 * b) % S if lengths else S for b in range(B)]
    got = kvbfp.decode_attention(cache, q, S, 0.1, seq_len_dev=dev_i32(np.asarray(lens)) if lengths else None)
    torch.cuda.synchronize()
    _oracle_units(cache, got, k, v, q, lens, n, 4, G, S, None, None, float(np.float32(0.1)), 0, torch.float32, [(0, 0), (B // 2, 3), (B - 1, 7)])


def _planned(dtype, p, n, B, Hkv, G, S, lengths, length):
    """Number of splits that a call over sequences of one length leaves partial results of (0: the split pass wrote the output)."""
    layout = kvbfp.make_layout(D, n, p, Hkv, B, S)
    cache = kvbfp.alloc_cache(layout, "cuda", fill=0)
    Hq = Hkv * G
    q = torch.zeros((B, Hq, D), dtype=dtype, device="cuda")
    ws = torch.zeros((kvbfp.decode_workspace_bytes(layout, Hq, S) + 4096,), dtype=torch.uint8, device="cuda")
    kvbfp.decode_attention(cache, q, S, 0.1, seq_len_dev=dev_i32(np.full(B, length)) if lengths else None, workspace=ws)
    torch.cuda.synchronize()
    if not bool(ws.any()):
        return 0
    for splits in range(1, 200):                      # all keys are 0: a split weighs as many tokens as it has
        rows = B * Hq * splits
        if rows * (D + 2) * 4 > ws.numel():
            break
        weight = ws.view(torch.float32)[rows * D:rows * (D + 2)].view(B, Hq, splits, 2)[..., 1]
        if bool((weight.sum(-1) == length).all()):
            return int((weight[0, 0] > 0).sum())
    return -1


# (8 kv-heads) between one and two splits, two and three workgroups per compute unit
@pytest.mark.parametrize("B,S,lengths,want", [
    (4, 4352, True, 16), (4, 9216, True, 16), (16, 1536, True, 4),          # 17, 36 tiles of 32 units, 6 of 128: two per compute unit
    (24, 1200, True, 3), (24, 3072, True, 2), (24, 3073, True, 4), (24, 4096, False, 2), (24, 4097, False, 4),      # 192 units: three where it pays
    (33, 1536, True, 0), (33, 1537, True, 2), (33, 2048, False, 0), (33, 2100, False, 2),
    (64, 3072, True, 0), (64, 3073, True, 2), (64, 4096, False, 0),
    (65, 4096, True, 0), (65, 4097, True, 2), (65, 4097, False, 0)])
def test_splits_of_the_plan(B, S, lengths, want):
    assert _planned(torch.float32, 4, 32, B, 8, 1, S, lengths, S) == want


@pytest.mark.parametrize("n,B,S,lengths", [(16, 24, 3073, True), (32, 24, 4097, False), (16, 40, 2400, True), (32, 130, 200, True), (64, 200, 700, False), (32, 33, 1536, True), (64, 33, 1537, True), (32, 64, 3073, True), (16, 48, 2100, False)])
def test_either_side_of_the_lines_of_the_plan(n, B, S, lengths):
    test_two_and_three_workgroups_per_compute_unit(n, B, S, lengths)
