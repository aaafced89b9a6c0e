"""Row-tiled GEMM against the oracle: every output tile, every pair of tile and
epilogue that the workloads dispatch, and K splits of 1 to 6, at row and column
counts around the tile edges, through prefill chunks of a given number of rows
(three prompts in one chunk, so row positions jump inside a tile), verify passes
and draft calls.  Which of them run on row tiles is the library's own plan."""
import ctypes as C

import numpy as np
import pytest

import synth
from oracle import model as om
from paper_2510_11331_amd import _lib
from paper_2510_11331_amd.engine import model_cfg
from sdcase import make_engine, run_gpu_steps, say

WIDE = synth.ModelShape(2, 1024, 8, 8, 11008, 1008, "bf16")
NARROW = synth.ModelShape(2, 512, 8, 1, 1408, 1008, "bf16")    # GQA: 640 QKV columns; 1008 logits end inside a tile
DRAFT = synth.ModelShape(1, 128, 2, 2, 256, 1008, "bf16")
CASES = [(WIDE, 65), (WIDE, 129), (WIDE, 161), (WIDE, 257), (WIDE, 330), (WIDE, 511), (WIDE, 700), (WIDE, 1030),
         (WIDE, 2049), (NARROW, 127), (NARROW, 700), (NARROW, 1030)]
# Largest error of a row over its largest logit, against the model with the
# same fp16 storage points: sums of another order move some operands to the
# neighbouring fp16 value (2^-11), at the four product inputs and the K/V and
# q roundings of two layers and the final norm: at most 2^-11 (2 x 6 + 1) / 2
BOUND = 2.0 ** -11 * 6.5


EPI = ("qkv", "kv", "resid", "gateup", "resid", "store")       # by SD_PROJ_*
DECODE = (_lib.SD_PROJ_QKV, _lib.SD_PROJ_O, _lib.SD_PROJ_GATEUP, _lib.SD_PROJ_DOWN, _lib.SD_PROJ_LM_HEAD)
PREFILL = (_lib.SD_PROJ_QKV, _lib.SD_PROJ_KV, _lib.SD_PROJ_O, _lib.SD_PROJ_GATEUP, _lib.SD_PROJ_DOWN)


def _config(shape, draft, **kw):
    c = _lib.Config()
    c.target, c.draft = model_cfg(shape), model_cfg(draft)
    c.max_slots = c.max_batch = kw.get("batch", 3)
    c.gamma_max, c.max_ctx, c.kv_block, c.temperature = kw.get("gamma", 1), 4096, 16, 1.0
    c.prefill_rows, c.kv_blocks_target, c.kv_blocks_draft = kw.get("prefill_rows", 256), 64, 64
    return c


def _plan(cfg, pass_, proj, rows):
    p = _lib.ProjPlan()
    _lib.check(_lib.lib().sd_plan_projection(C.byref(cfg), pass_, proj, rows, C.byref(p)), "sd_plan_projection")
    return p


def _row_tiled(cfg, pass_, rows):
    """(epilogue, tile, K split) of a pass's projections that run on row tiles."""
    plans = [(EPI[j], _plan(cfg, pass_, j, rows)) for j in (PREFILL if pass_ >= _lib.SD_PASS_PREFILL else DECODE)]
    return [(e, p.tile, p.ksplit) for e, p in plans if p.tile >= 0]


def _plans(shape, M, draft=DRAFT):
    """Those of a prefill chunk of M rows."""
    return _row_tiled(_config(shape, draft, prefill_rows=M), _lib.SD_PASS_PREFILL, M)


def test_cases_reach_every_tile():
    plans = [p for s, M in CASES for p in _plans(s, M)]
    assert {t for _, t, _ in plans} == set(range(11))
    assert {k for _, _, k in plans} >= {1, 2, 3, 4, 5, 6}


def test_dispatch_follows_the_grid():
    """The rules that move a projection between the skinny GEMM and the row tiles, on both sides of each: one round of
    skinny workgroups for 256 CUs (32 columns and 64 rows each; QKV up to 64 rows 16 columns), the weights from which
    a residual projection's larger K split pays, and the widths that balanced and 48-column tiles hold."""
    V, Q, O, GU, DOWN = (_lib.SD_PASS_VERIFY, _lib.SD_PROJ_QKV, _lib.SD_PROJ_O, _lib.SD_PROJ_GATEUP, _lib.SD_PROJ_DOWN)
    sh = lambda d, H, KV, F: synth.ModelShape(1, d, H, KV, F, 1008, "bf16")
    cases = [
        (sh(2048, 32, 16, 2048), Q, {64: 0, 65: 0, 128: 0, 129: 1}),       # 4096 columns: two row blocks are one round
        (sh(1408, 22, 22, 2112), Q, {48: 0, 49: 1, 65: 1, 128: 1}),        # 4224
        (sh(2048, 32, 16, 2048), GU, {64: 0, 65: 0, 128: 0, 129: 1}),      # 4096
        (sh(2048, 32, 16, 2112), GU, {49: 0, 64: 0, 65: 1, 128: 1}),       # 4224: one row block is one round still
        (sh(2048, 32, 16, 4160), GU, {32: 0, 48: 0, 49: 1, 64: 1}),        # 8320
        (sh(2048, 16, 16, 5632), O, {8: 0, 40: 0, 64: 0, 65: 1}),          # 4.2 M, 2048 columns: one round
        (sh(2304, 18, 18, 5632), O, {8: 0, 32: 0, 33: 1, 64: 1}),          # 5.3 M, 2304 columns: more
        (sh(2048, 16, 16, 7808), DOWN, {64: 0, 65: 1}),                    # 15.99 M weights
        (sh(2048, 16, 16, 7872), DOWN, {48: 0, 49: 1, 64: 1}),             # 16.1 M
        (sh(2048, 16, 16, 9728), DOWN, {16: 0, 17: 0, 48: 0, 49: 1}),      # 19.9 M
        (sh(2048, 16, 16, 9792), DOWN, {1: 1, 16: 1, 17: 1, 48: 1}),       # 20.05 M
        (sh(1024, 16, 16, 12288), GU, {1: 0, 48: 0, 49: 1}),               # 24576: the most balanced mode holds
        (sh(1024, 16, 16, 12352), GU, {1: 1, 32: 1, 48: 1}),
        (sh(1024, 16, 16, 16384), GU, {1: 0, 32: 0, 33: 1}),               # 32768
        (sh(4096, 32, 32, 64), Q, {1: 0, 48: 0, 49: 1}),                   # 12288
        (sh(4224, 33, 33, 64), Q, {1: 1, 48: 1}),                          # 12672
        (sh(5248, 41, 41, 64), Q, {1: 0, 16: 0, 17: 1}),                   # 15744
    ]
    for shape, proj, want in cases:
        c = _config(shape, DRAFT, batch=128)
        got = {rows: int(_plan(c, V, proj, rows).tile >= 0) for rows in want}
        assert got == want, (shape, proj, got, want)
    c = _config(synth.MODELS["tiny_target"].replace(vocab=1008), DRAFT, batch=128)
    assert all(_plan(c, V, p, r).tile < 0 for p in DECODE for r in (1, 64, 256))      # fp32 has no row tiles


def test_no_k_range_is_empty():
    """Every range of a K split holds at least one of its tile's stages, in all the passes of the workloads and of narrow
    models whose K is a few stages."""
    shapes = [(w.target, w.draft) for w in synth.WORKLOADS.values() if w.target.dtype == "bf16"]
    shapes += [(synth.ModelShape(2, d, d // 64, d // 64, F, 1008, "bf16"), DRAFT)
               for d, F in ((64, 64), (128, 128), (192, 448), (256, 320), (320, 2752), (640, 704), (832, 5440))]
    split = 0
    for t, d in shapes:
        c = _config(t, d, batch=128, prefill_rows=2048)
        for ps, most in ((_lib.SD_PASS_VERIFY, 256), (_lib.SD_PASS_DRAFT, 256), (_lib.SD_PASS_PREFILL, 2048),
                         (_lib.SD_PASS_PREFILL_DRAFT, 2048)):
            for rows in list(range(1, 257)) + list(range(257, most + 1, 7)):
                for proj in (_lib.SD_PROJ_O, _lib.SD_PROJ_DOWN):
                    p = _plan(c, ps, proj, rows)
                    if p.tile >= 0 and p.ksplit > 1:
                        stages = -(-p.K // (32 * p.ks))
                        assert (p.ksplit - 1) * -(-stages // p.ksplit) < stages, (t, ps, proj, rows, p.tile, p.ksplit)
                        split += 1
    assert split > 1000


@pytest.mark.gpu
@pytest.mark.parametrize("shape,rows", CASES, ids=lambda v: str(v) if isinstance(v, int) else f"d{v.d_model}")
def test_prefill_chunk_matches_oracle(shape, rows):
    say("row tiles", shape, rows, _plans(shape, rows))
    lens = [rows // 3 + 1, rows // 2 + 1]
    lens.append(rows - sum(lens) + 3)                          # prompt[:-1] of the three fills the chunk
    assert sum(n - 1 for n in lens) == rows
    prompts = synth.prompts(3, lens, shape.vocab)
    tw, dw = synth.model_weights(shape, 5), synth.model_weights(DRAFT, 6)
    eng = make_engine(shape, DRAFT, tw, dw, max_slots=3, max_batch=3, gamma_max=1, max_ctx=max(lens) + 16,
                      prefill_rows=rows)
    _, _, b, z = run_gpu_steps(eng, [0, 1, 2], prompts, 1, 1, 9, [0, 1, 2], keep_logits=True)
    drafts = b.draft_tok.cpu().numpy()
    assert eng.check_flags() == 0
    eng.close()
    ref = om.Model(shape, tw).sequence_logits([list(p) + [int(drafts[k, 0])] for k, p in enumerate(prompts)], 2)
    for k in range(3):
        for j in range(2):
            err = float(np.abs(z[0, k, j] - ref[k][j]).max() / np.abs(ref[k][j]).max())
            assert err < BOUND, (k, j, err)


def _verify(shape, B, gamma, draft=DRAFT):
    say("row tiles, verify", shape, B, gamma, draft)
    prompts = synth.prompts(B, [5 + k % 7 for k in range(B)], shape.vocab)
    tw, dw = synth.model_weights(shape, 5), synth.model_weights(draft, 6)
    eng = make_engine(shape, draft, tw, dw, max_slots=B, max_batch=B, gamma_max=gamma, max_ctx=64, prefill_rows=256)
    _, _, b, z = run_gpu_steps(eng, list(range(B)), prompts, gamma, 1, 9, list(range(B)), keep_logits=True)
    drafts, q = b.draft_tok.cpu().numpy(), b.q.cpu().numpy().astype(np.float64)
    assert eng.check_flags() == 0
    eng.close()
    seqs = [list(p) + [int(t) for t in drafts[k]] for k, p in enumerate(prompts)]
    ref = om.Model(shape, tw).sequence_logits(seqs, gamma + 1)
    zd = om.Model(draft, dw).sequence_logits([sq[:-1] for sq in seqs], gamma)
    for k in range(B):
        for i in range(gamma):
            dlog = np.log(q[k, i]) - zd[k][i]
            assert np.ptp(dlog) < 2 * BOUND * np.abs(zd[k][i]).max(), (k, i)
    for k in range(B):
        for j in range(gamma + 1):
            err = float(np.abs(z[0, k, j] - ref[k][j]).max() / np.abs(ref[k][j]).max())
            assert err < BOUND, (k, j, err)


LONG_FFN = synth.ModelShape(1, 1024, 8, 8, 20480, 1008, "bf16")   # gate/up past balanced mode, 21 M down projection
WIDE_QKV = synth.ModelShape(1, 4224, 33, 33, 512, 1008, "bf16")    # 12672 QKV columns


SMALL_PASSES = [(LONG_FFN, 1, 1), (LONG_FFN, 1, 4), (LONG_FFN, 3, 5), (LONG_FFN, 16, 2), (LONG_FFN, 7, 6), (LONG_FFN, 16, 3),
                (WIDE_QKV, 1, 4), (WIDE_QKV, 8, 5), (WIDE_QKV, 13, 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,B,gamma", SMALL_PASSES,
                         ids=lambda v: str(v) if isinstance(v, int) else f"d{v.d_model}")
def test_small_pass_of_wide_projections_matches_oracle(shape, B, gamma):
    """Passes of up to one 64-row block whose wide projections run on row tiles (2 to 65 rows)."""
    _verify(shape, B, gamma)


ROUTED = [(synth.ModelShape(1, 2048, 32, 16, 2112, 1008, "bf16"), 13, 4),   # 65 rows: QKV skinny, gate/up on row tiles
          (synth.ModelShape(1, 1536, 24, 24, 512, 1008, "bf16"), 7, 4),     # 35: O
          (synth.ModelShape(1, 1536, 24, 24, 512, 1008, "bf16"), 10, 4),    # 50: QKV and O
          (synth.ModelShape(1, 1024, 16, 16, 14336, 1008, "bf16"), 1, 4),   # 5: gate/up of 28672 columns
          (synth.ModelShape(1, 1024, 16, 16, 14336, 1008, "bf16"), 7, 4),   # 35
          (synth.ModelShape(1, 5248, 41, 41, 64, 1008, "bf16"), 3, 4),      # 15: O; QKV of 15744 columns skinny
          (synth.ModelShape(1, 5248, 41, 41, 64, 1008, "bf16"), 4, 4)]      # 20: QKV and O


@pytest.mark.gpu
@pytest.mark.parametrize("shape,B,gamma", ROUTED, ids=lambda v: str(v) if isinstance(v, int) else f"d{v.d_model}")
def test_both_sides_of_the_dispatch_match_oracle(shape, B, gamma):
    assert _row_tiled(_config(shape, DRAFT, batch=B, gamma=gamma), _lib.SD_PASS_VERIFY, B * (gamma + 1))
    _verify(shape, B, gamma)


BATCHED = [(13, 4), (24, 4), (33, 7), (70, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,gamma", BATCHED)
def test_batched_verify_matches_oracle(B, gamma):
    """65 to 264 verified rows: K-split residual projections, an LM head whose last column tile is partial, values of
    several tasks in one row tile (and, in the 140 rows of the last case's first draft call, every other row inactive)."""
    _verify(NARROW, B, gamma)


# K = 64 (mod 128) in every projection: the last stage of the tiles of four
# k-steps per stage (6, 8 and 10: 128 x 64, 96 x 64, 64 x 64) is half full
ODD320 = synth.ModelShape(2, 320, 5, 5, 2752, 1008, "bf16")
ODD832 = synth.ModelShape(2, 832, 13, 13, 5440, 1008, "bf16")
ODD192 = synth.ModelShape(2, 192, 3, 1, 64, 1008, "bf16")          # down projection of two k-steps: half a stage
ODD_LONG = synth.ModelShape(1, 832, 13, 13, 24128, 1008, "bf16")   # 20 M down projection: row tiles from one row on
ODD_DRAFT = synth.ModelShape(1, 320, 5, 5, 576, 1008, "bf16")
ODD_CASES = [(ODD320, 65), (ODD320, 512), (ODD320, 1500), (ODD320, 2049), (ODD832, 100), (ODD832, 257), (ODD832, 320),
             (ODD832, 640), (ODD832, 2049), (ODD192, 127)]


def test_odd_k_cases_reach_every_four_step_tile():
    plans = {p for s, M in ODD_CASES for p in _plans(s, M)}
    assert {t for _, t, _ in plans} >= {6, 8, 10}
    assert {(t, k > 1) for e, t, k in plans if e == "resid"} >= {(6, True), (8, True), (10, True), (6, False), (10, False)}


@pytest.mark.gpu
@pytest.mark.parametrize("shape,rows", ODD_CASES, ids=lambda v: str(v) if isinstance(v, int) else f"d{v.d_model}")
def test_prefill_chunk_of_odd_k_matches_oracle(shape, rows):
    test_prefill_chunk_matches_oracle(shape, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,B,gamma", [(ODD832, 13, 4), (ODD832, 70, 1), (ODD320, 33, 7), (ODD_LONG, 1, 1),
                                           (ODD_LONG, 8, 4), (ODD_LONG, 12, 4)],
                         ids=lambda v: str(v) if isinstance(v, int) else f"d{v.d_model}")
def test_verify_and_draft_of_odd_k_match_oracle(shape, B, gamma):
    """Verify passes of 2 to 264 rows and (B > 32) draft calls of more than one 64-row block."""
    _verify(shape, B, gamma, ODD_DRAFT)


def _shape(d, H, KV, F, layers=2, vocab=1008):
    return synth.ModelShape(layers, d, H, KV, F, vocab, "bf16")


# The pairs of tile and epilogue of the 7B-, 13B- and small workloads that the cases above leave out, at narrower widths
PAIR_PREFILL = [(_shape(1024, 8, 8, 512), 801), (_shape(1024, 8, 8, 512), 1281), (_shape(2048, 16, 16, 512), 900),
                (_shape(2048, 16, 16, 512), 1540), (_shape(2048, 16, 16, 512), 2049), (_shape(2048, 16, 16, 5120), 801),
                (_shape(2176, 17, 17, 512), 400), (_shape(2176, 17, 17, 5120), 1160), (_shape(3072, 24, 24, 512), 1601),
                (_shape(3072, 24, 24, 512), 1930), (_shape(3072, 24, 24, 5120), 1030), (_shape(4096, 32, 32, 512), 260),
                (_shape(4096, 32, 32, 512), 2049)]
WIDE_HEAD = _shape(128, 2, 2, 512, 1, 32000)
PAIR_VERIFY = [(17, 5), (19, 6), (26, 6), (33, 7), (49, 7), (65, 7)]          # 102 to 520 rows of 32000 logits


def _pairs(cfg, pass_, rows):
    return {(t, "partial sums" if k > 1 else e) for e, t, k in _row_tiled(cfg, pass_, rows)}


def test_cases_cover_the_workloads():
    """Every (tile, epilogue) that a pass of the bf16 workloads runs on, at any number of rows, is in a GPU case."""
    V, D, P, PD = _lib.SD_PASS_VERIFY, _lib.SD_PASS_DRAFT, _lib.SD_PASS_PREFILL, _lib.SD_PASS_PREFILL_DRAFT
    want = set()
    for w in synth.WORKLOADS.values():
        if w.target.dtype == "bf16":
            c = _config(w.target, w.draft, batch=64, gamma=8, prefill_rows=2048)
            for ps, n in ((V, 576), (D, 128), (P, 2048), (PD, 2048)):
                want |= set().union(*(_pairs(c, ps, rows) for rows in range(1, n + 1)))
    have = set()
    for shape, rows in CASES + ODD_CASES + PAIR_PREFILL:
        have |= _pairs(_config(shape, DRAFT, prefill_rows=rows), P, rows)
    for shape, B, gamma in (SMALL_PASSES + ROUTED + [(NARROW, B, g) for B, g in BATCHED]
                            + [(WIDE_HEAD, B, g) for B, g in PAIR_VERIFY]):
        c = _config(shape, DRAFT.replace(vocab=shape.vocab), batch=B, gamma=gamma)
        have |= _pairs(c, V, B * (gamma + 1)) | _pairs(c, D, B) | _pairs(c, D, 2 * B)
    assert len(want) >= 50 and want <= have, sorted(want - have)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,rows", PAIR_PREFILL, ids=lambda v: str(v) if isinstance(v, int) else f"d{v.d_model}-F{v.d_ffn}")
def test_prefill_chunk_of_other_tiles_matches_oracle(shape, rows):
    test_prefill_chunk_matches_oracle(shape, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("B,gamma", PAIR_VERIFY)
def test_wide_head_on_row_tiles_matches_oracle(B, gamma):
    _verify(WIDE_HEAD, B, gamma, DRAFT.replace(vocab=WIDE_HEAD.vocab))
