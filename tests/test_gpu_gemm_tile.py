"""GPU: the many-row decoder GEMM (gemm_tile_kernel) through
draft_verify_step: against the float64 oracle (64 x 64 tiles for the layer,
every tile size for the head; rows and columns that end inside a tile; K with
one and with four logical splits), its fused top-1 against the logits, and at
every tile size and epilogue its rows bit for bit against the few-row
kernels'."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decode as od
from oracle.model import OracleModel
from paper_2609_26638_amd import dvs, synth
from tests.gpu_util import max_rel_err, to_dev

pytestmark = pytest.mark.gpu


def _model(H, Hq, Hkv, D, ffn, V, S, nc, nm):
    w = synth.make_model_weights(11, V, H, Hq, Hkv, D, 1, ffn, std=0.08)
    lens = [(37 + 61 * s) % 200 for s in range(S)]
    ai = synth.make_attn_inputs(11, S, lens, nc, nm, Hq, Hkv, D, "bf16", std=0.5, scatter=True,
                                extra_pages=4 * S)
    rng = np.random.default_rng(5)
    ai.state.boundary[:] = rng.integers(0, V, size=S)
    ai.state.draft[:] = rng.integers(0, V, size=ai.state.draft.shape)
    return w, ai


def _shift(dm, shift):
    """Every weight starts ``shift`` elements into another tensor."""
    def moved(t):
        buf = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
        return buf[shift:].view(t.shape).copy_(t)

    for n in ("embed", "g_final", "lm_head"):
        setattr(dm, n, moved(getattr(dm, n)))
        setattr(dm.desc, n, getattr(dm, n).data_ptr())
    for l, t in enumerate(dm.keep):
        for n in t:
            t[n] = moved(t[n])
            setattr(dm.layers[l], n, t[n].data_ptr())
            assert t[n].data_ptr() % 16 == shift * 2 % 16


def _step(w, ai, host, nc, nm, shift=0):
    """(logits [S, R, V], top-1 with the logits, top-1 without)"""
    S, R = host.kv_len.shape[0], nc + nm
    lg = torch.empty((S, R, w.V), dtype=torch.float32, device="cuda")
    ams = []
    for logits in (lg, None):
        dm = dvs.DeviceModel(w, [to_dev(ai.k_pool, "bf16")], [to_dev(ai.v_pool, "bf16")], "bf16")
        if shift:
            _shift(dm, shift)
        st = dvs.DeviceState(host)
        am = torch.empty((S, R), dtype=torch.int32, device="cuda")
        dvs.draft_verify_step(dm, st, nc, nm, logits_out=logits, argmax_out=am)
        assert int(st.err.item()) == 0
        ams.append(am.cpu().numpy())
    return lg.cpu().numpy(), ams[0], ams[1]


# (hidden, heads, kv heads, head dim, ffn, vocab, sequences, causal, mask):
# 520 rows: 64 x 64 tiles for the layer, 128 x 256 for the head (odd vocab);
# the same rows with a head of 128 x 128 tiles; 257 rows with one K split and
# a last column block of 8; 3 rows with one K split and K of three chunks.
@pytest.mark.parametrize("H,Hq,Hkv,D,ffn,V,S,nc,nm", [
    (256, 4, 2, 64, 512, 33001, 13, 20, 20),
    (256, 2, 1, 128, 512, 5000, 13, 40, 0),
    (320, 5, 1, 64, 448, 1000, 1, 257, 0),
    (192, 2, 2, 96, 192, 515, 1, 2, 1),
])
def test_many_row_step_matches_oracle(H, Hq, Hkv, D, ffn, V, S, nc, nm):
    w, ai = _model(H, Hq, Hkv, D, ffn, V, S, nc, nm)
    rnd = lambda a: synth.bf16_to_f32(synth.f32_to_bf16_bits(a))
    wb = dataclasses.replace(w, **{
        f.name: [rnd(a) for a in v] if isinstance(v, list) else rnd(v)
        for f in dataclasses.fields(w)
        if isinstance(v := getattr(w, f.name), (list, np.ndarray))})
    om = OracleModel(wb, [synth.bf16_to_f32(ai.k_pool)], [synth.bf16_to_f32(ai.v_pool)])
    tok = np.full((S, nc + nm), V, np.int64)
    tok[:, 0] = ai.state.boundary
    tok[:, 1:nc] = ai.state.draft[:, :nc - 1]
    ref = om.forward(om.embed[tok], ai.state.copy(), nc, nm)
    lg, am, am2 = _step(w, ai, ai.state, nc, nm)
    # bf16 activations between the layer's kernels: a few 1e-3 of the largest
    # logit each, as for the few-row steps
    assert max_rel_err(lg.astype(np.float64), ref) <= 5e-2
    np.testing.assert_array_equal(am, od.top1_rows(lg.astype(np.float64)))
    np.testing.assert_array_equal(am2, am)


# Sequences, causal and mask rows each, hidden, heads, kv heads, head dim, ffn,
# vocab.  520 rows: 64 x 64 tiles for the layer at every head dim (the rotary
# epilogue), alone 40 rows or the narrow blocks' 10, the head in 128 x 256
# tiles, alone in the column-split kernel; 240 rows: gate|up in 128 x 64 tiles
# and Q|K|V in the row-split kernel; 1040 rows: Q|K|V and gate|up in 128 x 128
# tiles; 2200 rows: the residual in those; 8320 rows: all in 128 x 256 tiles,
# the last ones part empty.
@pytest.mark.parametrize("S,nc,nm,H,Hq,Hkv,D,ffn,V", [
    (13, 20, 20, 256, 4, 2, 64, 512, 33001),
    (13, 20, 20, 256, 4, 2, 96, 512, 5000),
    (52, 5, 5, 256, 2, 1, 128, 512, 5000),
    (6, 20, 20, 256, 16, 4, 96, 4096, 33001),
    (26, 20, 20, 256, 16, 4, 96, 1152, 5000),
    (55, 20, 20, 1536, 4, 2, 64, 256, 1000),
    (208, 20, 20, 1024, 4, 2, 64, 256, 1000),
])
def test_rows_equal_the_few_row_kernels(S, nc, nm, H, Hq, Hkv, D, ffn, V):
    """All sequences in one call, then each of three alone, with the logits
    and with the fused top-1 alone."""
    w, ai = _model(H, Hq, Hkv, D, ffn, V, S, nc, nm)
    lg, am, top = _step(w, ai, ai.state, nc, nm)
    np.testing.assert_array_equal(top, am)
    for s in (0, S // 2, S - 1):
        h = ai.state.copy()
        for f in ("kv_len", "page_table", "num_pages", "boundary", "draft", "out_tokens",
                  "out_count", "finished"):
            setattr(h, f, getattr(h, f)[s:s + 1].copy())
        one, am1, top1 = _step(w, ai, h, nc, nm)
        np.testing.assert_array_equal(one[0], lg[s])
        np.testing.assert_array_equal(am1[0], am[s])
        np.testing.assert_array_equal(top1[0], am[s])


# Weights at element alignment, of one and of four K splits, few rows and many.
@pytest.mark.parametrize("H,Hq,Hkv,D,ffn,V,S,nc,nm,shift", [
    (320, 5, 1, 64, 448, 1000, 1, 257, 0, 1),
    (192, 2, 2, 96, 192, 515, 2, 2, 1, 4),
    (256, 2, 1, 128, 512, 5000, 13, 40, 0, 1),
    (256, 4, 2, 64, 512, 33001, 2, 20, 20, 2),
])
def test_weights_at_element_alignment(H, Hq, Hkv, D, ffn, V, S, nc, nm, shift):
    w, ai = _model(H, Hq, Hkv, D, ffn, V, S, nc, nm)
    ref = _step(w, ai, ai.state, nc, nm)
    got = _step(w, ai, ai.state, nc, nm, shift)
    for a, b in zip(got, ref):
        np.testing.assert_array_equal(a, b)
