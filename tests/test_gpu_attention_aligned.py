"""GPU: aligned attention chunks shared over workgroups.  An item's chunks run
in one workgroup or in many, the window is appended by the attention launch
(one row tile) or by one of its own (several), and chunks past the keys a row
tile sees are skipped: against the oracle, and every sequence of a batch bit
for bit against the same sequence alone (which splits its chunks otherwise)."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2609_26638_amd import dvs, synth
from tests.gpu_util import dev_attn, max_rel_err, to_f64

pytestmark = pytest.mark.gpu


def _call(d, s, nc, nm, group, scale, chunk):
    sl = slice(s, s + 1) if s is not None else slice(None)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    kp, vp = d["k_pool"].clone(), d["v_pool"].clone()
    out = dvs.attn_hybrid_block_grouped(d["q"][sl], d["k_new"][sl], d["v_new"][sl], kp, vp,
                                        d["page_table"][sl], d["kv_len"][sl], nc, nm, group, scale,
                                        err=err, chunk_keys=chunk)
    assert int(err.item()) == 0
    return out, kp, vp


# (lens, causal, mask, group, heads, kv heads, head dim, chunk): a prefill (no
# cache, many row tiles, each seeing its own prefix); a batch of many items
# (runs of several chunks per workgroup) whose row tiles end inside a wave; one
# row tile with a window over a chunk's edge; mask groups that skip the tiles
# of the groups before; one AR row at the edges of tiles and chunks.
@pytest.mark.parametrize("lens,nc,nm,group,Hq,Hkv,D,chunk", [
    ([0, 0], 397, 7, 0, 8, 2, 96, 128),
    ([700, 65, 1023, 0, 311, 64, 900, 128] * 6, 33, 7, 0, 16, 4, 64, 64),
    ([250, 255, 256, 640, 63], 13, 13, 0, 8, 2, 128, 256),
    ([500, 190], 8, 64, 8, 16, 4, 96, 128),
    ([500, 190, 3], 12, 144, 12, 8, 2, 128, 64),
    ([0, 63, 64, 255, 256, 1500], 1, 0, 0, 4, 1, 96, 256),
    ([700, 65, 0, 1000], 40, 24, 0, 16, 4, 64, 128),     # two row tiles, each appending
    ([300, 17, 64], 150, 50, 0, 4, 4, 64, 64),           # two row tiles, an append launch
    # 516 items of four row tiles: one workgroup streams all of an item's chunks
    # (up to five) and merges its own partials; the XCDs' last run is short
    ([0, 500, 250, 401] + [(83 * s) % 520 for s in range(39)], 60, 40, 0, 12, 3, 64, 128),
    # 516 items again, one of 87 chunks: its page ids are staged a second time
    # 256 tiles on, inside a chunk of three tiles
    ([16500, 200, 0, 64] + [30] * 125, 2, 1, 0, 8, 4, 64, 192),
])
def test_aligned_chunks(lens, nc, nm, group, Hq, Hkv, D, chunk):
    S = len(lens)
    ai = synth.make_attn_inputs(3, S, lens, nc, nm, Hq, Hkv, D, "bf16", std=1.0, scatter=True)
    d = dev_attn(ai)
    out, kp, vp = _call(d, None, nc, nm, group, ai.scale, chunk)
    for s in sorted({0, 1, S - 1}):
        one, _, _ = _call(d, s, nc, nm, group, ai.scale, chunk)
        assert torch.equal(one[0], out[s]), s
    n = min(S, 4)
    k_ref, v_ref = ai.as_f64("k_pool"), ai.as_f64("v_pool")
    ref = oa.attn_hybrid_block(ai.as_f64("q")[:n], ai.as_f64("k_new")[:n], ai.as_f64("v_new")[:n],
                               k_ref, v_ref, ai.state.page_table[:n], ai.state.kv_len[:n], nc, nm,
                               ai.scale, group=group)
    assert max_rel_err(to_f64(out[:n]), ref) <= 2e-2
    # the window reached its slots and nothing else changed
    for s in range(n):
        held = ai.state.page_table[s][:(lens[s] + nc + nm + 15) // 16]
        np.testing.assert_array_equal(to_f64(kp)[held], k_ref[held])
        np.testing.assert_array_equal(to_f64(vp)[held], v_ref[held])


# The merge by a launch of its own (many output elements, or many segments)
# and by the last workgroup, in both splits, at every wave count of the
# balanced one; one item whole and one split in the same call.
@pytest.mark.parametrize("lens,R,Hq,Hkv,D,chunk", [
    ([1500, 30], 8, 16, 4, 128, 0),      # 32 rows, one wave, 16 segments
    ([1500, 30, 700], 16, 8, 2, 96, 0),  # 64 rows, two waves
    ([4000, 0], 30, 16, 4, 64, 0),       # 120 rows, four waves
    ([900, 63], 25, 16, 4, 128, 64),     # 100 rows, aligned
    ([2000, 5], 1, 8, 2, 64, 64),        # 4 rows in 32 chunks
    ([300] * 24, 3, 8, 4, 64, 64),       # 6 rows, count-in
])
def test_merge(lens, R, Hq, Hkv, D, chunk):
    ai = synth.make_attn_inputs(9, len(lens), lens, R, 0, Hq, Hkv, D, "bf16", std=1.0, scatter=True)
    d = dev_attn(ai)
    ws = dvs.Workspace(256)
    outs = []
    for _ in range(3):   # the same workspace: whatever a call leaves in it
        outs.append(dvs.attn_hybrid_block(d["q"], d["k_new"], d["v_new"], d["k_pool"], d["v_pool"],
                                          d["page_table"], d["kv_len"], R, 0, ai.scale,
                                          workspace=ws, chunk_keys=chunk))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    n = min(len(lens), 3)
    ref = oa.attn_hybrid_block(ai.as_f64("q")[:n], ai.as_f64("k_new")[:n], ai.as_f64("v_new")[:n],
                               ai.as_f64("k_pool"), ai.as_f64("v_pool"), ai.state.page_table[:n],
                               ai.state.kv_len[:n], R, 0, ai.scale)
    assert max_rel_err(to_f64(outs[0][:n]), ref) <= 2e-2


# A row's bits do not depend on who merges its chunks: a launch (alone), the
# last workgroup to count in (20 sequences, seven workgroups per item), or the
# only workgroup (130 sequences).
@pytest.mark.parametrize("D", [64, 96, 128])
def test_merges_have_the_same_bits(D):
    lens = [700, 641, 900, 577] + [(37 * s) % 800 for s in range(126)]
    ai = synth.make_attn_inputs(19, len(lens), lens, 1, 0, 8, 4, D, "bf16", std=1.0, scatter=True)
    d = dev_attn(ai)
    outs = []
    for n in (1, 20, 130):
        a = {f: x if f.endswith("pool") else x[:n] for f, x in d.items()}
        outs.append(dvs.attn_hybrid_block(**a, n_causal=1, n_mask=0, softmax_scale=ai.scale,
                                          chunk_keys=64))
    assert torch.equal(outs[0], outs[1][:1]) and torch.equal(outs[1], outs[2][:20])
    for s in (1, 2, 3):   # and the others alone
        a = {f: x if f.endswith("pool") else x[s:s + 1] for f, x in d.items()}
        one = dvs.attn_hybrid_block(**a, n_causal=1, n_mask=0, softmax_scale=ai.scale, chunk_keys=64)
        assert torch.equal(one[0], outs[2][s]), s


class _NeverCleared(dvs.Workspace):
    def prepare(self, nbytes, shape):
        assert nbytes <= self.nbytes
        return self


# A workspace zeroed once serves other shapes whose counters lie in those of
# the first: a call of many items whose chunks stay in one workgroup (it counts
# nothing in), one merged by a launch (balanced, with its segment table), then
# a small one that counts in.
def test_shapes_share_the_workspace_counters():
    many = synth.make_attn_inputs(21, 8, [300, 64, 200, 5, 0, 17, 0, 90], 512, 0, 16, 4, 64, "bf16",
                                  std=1.0, scatter=True)
    split = synth.make_attn_inputs(22, 4, [1500, 30, 700, 64], 30, 0, 16, 4, 64, "bf16", std=1.0,
                                   scatter=True)
    small = synth.make_attn_inputs(23, 2, [500, 190], 3, 0, 8, 4, 64, "bf16", std=1.0, scatter=True)
    calls = [(many, 128), (small, 128), (split, 0), (small, 128), (many, 128), (split, 0)]

    def call(ai, chunk, ws):
        d = dev_attn(ai)
        nc = ai.q.shape[1]
        return dvs.attn_hybrid_block(d["q"], d["k_new"], d["v_new"], d["k_pool"], d["v_pool"],
                                     d["page_table"], d["kv_len"], nc, 0, ai.scale, workspace=ws,
                                     chunk_keys=chunk)

    ws = _NeverCleared(1 << 28)
    for i, (ai, chunk) in enumerate(calls):
        own = call(ai, chunk, None)
        assert torch.equal(call(ai, chunk, ws), own), i


def test_more_sequences_than_a_grid_dimension():
    """65,600 equal sequences of two row tiles: the append launch holds them all."""
    S, R, Hq, Hkv, D, pages = 65600, 65, 2, 1, 64, 5
    g = torch.Generator(device="cuda").manual_seed(5)

    def same(*shape):
        x = torch.randn(1, *shape, generator=g, device="cuda").to(torch.bfloat16)
        return x.expand(S, *shape).contiguous()

    q, kn, vn = same(R, Hq, D), same(R, Hkv, D), same(R, Hkv, D)
    kp = torch.zeros(S * pages, Hkv, 16, D, dtype=torch.bfloat16, device="cuda")
    vp = torch.zeros(S * pages, Hkv, D, 16, dtype=torch.bfloat16, device="cuda")
    pt = torch.arange(S * pages, dtype=torch.int32, device="cuda").view(S, pages)
    lens = torch.zeros(S, dtype=torch.int32, device="cuda")
    out = dvs.attn_hybrid_block(q, kn, vn, kp, vp, pt, lens, R, 0, D ** -0.5, chunk_keys=128)
    one = dvs.attn_hybrid_block(q[:1], kn[:1], vn[:1], torch.zeros_like(kp[:pages]),
                                torch.zeros_like(vp[:pages]), pt[:1], lens[:1], R, 0, D ** -0.5,
                                chunk_keys=128)
    assert torch.equal(out, one.expand_as(out))
    k = kp.view(S, pages * 16, Hkv, D)[:, :R]
    assert torch.equal(k, kn)
