"""Attention against the oracle: the query-tile and key-group arrangements of the
16-bit decode kernel, the prefill kernel with its lazily raised maximum, and the
merge of the fp32 kernel's key splits."""
import math

import numpy as np
import pytest

import synth
from oracle import model as om
from sdcase import make_engine, run_gpu_steps, say

GQA = synth.ModelShape(1, 256, 4, 1, 512, 1008, "bf16")        # hd 64, 4 query heads per kv head
# Largest error of a row over its largest logit, against the model with the
# same fp16 storage points: 2^-11 at the operand roundings of one layer (normed
# row, q, K/V, attention output, normed row, SwiGLU output, final norm), where
# another order of summation can pick the neighbouring fp16 value
BOUND = 2.0 ** -11 * 7


def _compare(shape, dshape, prompts, gamma, tw=None, bound=BOUND, **kw):
    B = len(prompts)
    tw, dw = tw or synth.model_weights(shape, 5), synth.model_weights(dshape, 6)
    eng = make_engine(shape, dshape, tw, dw, max_slots=B, max_batch=B, gamma_max=gamma,
                      max_ctx=max(len(p) for p in prompts) + 2 * gamma + 16, **kw)
    _, _, b, z = run_gpu_steps(eng, list(range(B)), prompts, gamma, 1, 9, list(range(B)), keep_logits=True)
    drafts = b.draft_tok.cpu().numpy()
    assert eng.check_flags() == 0
    eng.close()
    ref = om.Model(shape, tw).sequence_logits([list(p) + [int(t) for t in drafts[k]] for k, p in enumerate(prompts)],
                                              gamma + 1)
    for k in range(B):
        for j in range(gamma + 1):
            err = float(np.abs(z[0, k, j] - ref[k][j]).max() / np.abs(ref[k][j]).max())
            assert err < bound, (k, j, err)


@pytest.mark.gpu
@pytest.mark.parametrize("gamma", [4, 8, 15])
@pytest.mark.parametrize("length", [6400, 700])
def test_query_tiles_of_grouped_heads(gamma, length):
    """20, 36 and 64 query vectors (2, 3 and 4 tiles) over 12 key splits: 6400 keys give every split more than the
    512 keys from which a wave takes several tiles, 700 do not; the second task ends inside a 32-key step."""
    say("query tiles", gamma, length)
    draft = synth.ModelShape(1, 128, 2, 2, 256, 1008, "bf16")
    _compare(GQA, draft, synth.prompts(2, [length, length - 99], GQA.vocab), gamma, prefill_rows=2048)


MHA128 = synth.ModelShape(2, 256, 2, 2, 512, 1008, "bf16")     # hd 128
GQA6 = synth.ModelShape(2, 384, 6, 1, 512, 1008, "bf16")       # hd 64, 6 query heads per kv head (21-row blocks)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [GQA.replace(n_layers=2), MHA128, GQA6], ids=["gqa4_hd64", "mha_hd128", "gqa6_hd64"])
@pytest.mark.parametrize("lens,rows", [((2, 18, 33, 65, 66), 2048), ((130, 129, 1), 100), ((700, 321), 512)])
def test_prefill_attention_matches_oracle(shape, lens, rows):
    """Prefill rows of several tasks in one chunk, chunks that start inside a task and inside a row block, key counts
    around the 16-key blocks and 64-key stages; slots reused after a longer task (values past the last key are stale)."""
    say("prefill attention", shape, lens, rows)
    draft = synth.ModelShape(1, 128, 2, 2, 256, 1008, "bf16")
    _compare(shape, draft, synth.prompts(len(lens), list(lens), shape.vocab), 2, prefill_rows=rows)


@pytest.mark.gpu
@pytest.mark.parametrize("gamma", [4, 8])
def test_query_tiles_of_large_grids(gamma):
    """1024 (task, kv head) items, the four-wave form, with key ranges on both sides of 512."""
    say("query tiles, large grid", gamma)
    shape = synth.ModelShape(1, 2048, 32, 8, 512, 1008, "bf16")
    draft = synth.ModelShape(1, 128, 2, 2, 256, 1008, "bf16")
    lens = [600 if k in (0, 77) else 515 - gamma if k == 5 else 3 + k % 40 for k in range(128)]
    _compare(shape, draft, synth.prompts(128, lens, shape.vocab), gamma, prefill_rows=2048)


# Scores far apart and rising along the keys.  All embeddings share a direction and the rotary frequencies past the
# first are ~0, so a key's score is nearly the same for every query; wq and wk are scaled until scores span more than
# 40 in log2 units, against the 8 from which the prefill kernel raises its running maximum and rescales.
RAISE, SCALE = 8.0, 12.0
PEAKED = [synth.ModelShape(2, 256, 4, 1, 512, 1008, "bf16", rope_theta=1e30),
          synth.ModelShape(2, 256, 2, 2, 512, 1008, "bf16", rope_theta=1e30)]


def _peaked_weights(shape):
    w = dict(synth.model_weights(shape, 5))
    f32 = synth.bf16_bits_to_f32
    common = np.random.default_rng(9).normal(0.0, 0.04, shape.d_model).astype(np.float32)
    w["embed"] = synth.bf16_bits(f32(w["embed"]) + common)
    for n in ("l0.wq", "l0.wk"):
        w[n] = synth.bf16_bits(f32(w[n]) * np.float32(SCALE))
    return w


def _layer0(shape, w, toks):
    m = om.Model(shape, w)
    h = m.r(om.rmsnorm(m.ops["embed"][toks], m.ops["l0.attn_norm"], shape.rms_eps))
    pos, hd = np.arange(len(toks)), shape.head_dim
    q = om.rope((h @ m.ops["l0.wq"].T).reshape(-1, shape.n_heads, hd), pos, shape.rope_theta)
    k = m.r(om.rope((h @ m.ops["l0.wk"].T).reshape(-1, shape.n_kv_heads, hd), pos, shape.rope_theta))
    return q, k


def _peaked_prompts(shape, w, n):
    """Random tokens in the order of their layer-0 score for head 0: rising, falling, and as drawn."""
    toks = synth.prompts(1, n, shape.vocab)[0]
    q, k = _layer0(shape, w, toks)
    order = np.argsort(k[:, 0] @ q[:, 0].mean(0))
    return [toks[order], toks[order[::-1]], toks]


def _scores(shape, w, toks, head):
    q, k = _layer0(shape, w, toks)
    s = q[:, head] @ k[:, head * shape.n_kv_heads // shape.n_heads].T / math.sqrt(shape.head_dim) / math.log(2.0)
    return np.where(np.tri(len(toks), dtype=bool), s, -np.inf)


def test_peaked_prompts_raise_the_maximum():
    """With the rising prompt, rows past the first few hundred raise the maximum in three and more 32-key steps after
    the first, beginning with different rows of a 16-query tile and different quarters of a step."""
    for shape in PEAKED:
        w = _peaked_weights(shape)
        s = _scores(shape, w, _peaked_prompts(shape, w, 700)[0], 0)
        assert np.ptp(s[-1]) > 40 and np.abs(s[np.isfinite(s)]).max() < 90
        rows, quarters = set(), set()
        for t in range(400, 688, 16):                            # the 16 queries of a tile share their raises
            m, raises = np.full(16, -1e30), 0
            for kb in range(0, t + 16, 32):
                x = s[t:t + 16, kb:kb + 32]
                over = np.argwhere(x > m[:, None] + RAISE)
                if len(over):
                    m = np.maximum(m, x.max(1))
                    if kb:
                        raises += 1
                        rows |= set(over[:, 0].tolist())
                        quarters |= set((over[:, 1] % 16 // 4).tolist())
            assert raises >= 3, (shape, t, raises)
        assert len(rows) > 8 and quarters == {0, 1, 2, 3}


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [2100, 96], ids=["one_chunk", "chunks_of_96"])
@pytest.mark.parametrize("shape", PEAKED, ids=["gqa4_hd64", "mha_hd128"])
def test_prefill_attention_of_peaked_scores_matches_oracle(shape, rows):
    """A key rounded to the neighbouring fp16 value (2^-11 of it) moves its score, up to 90 log2 units, by 2^-11 of
    itself, and p by as much in natural units; the rest as for the other tests here."""
    say("peaked prefill attention", shape, rows)
    draft = synth.ModelShape(1, 128, 2, 2, 256, 1008, "bf16")
    w = _peaked_weights(shape)
    _compare(shape, draft, _peaked_prompts(shape, w, 700), 2, tw=w, bound=BOUND + 2.0 ** -11 * 90 * math.log(2.0),
             prefill_rows=rows)


@pytest.mark.gpu
@pytest.mark.parametrize("hd", [64, 128])
def test_fp32_key_splits_match_oracle(hd):
    """12 key splits of 128 positions each: full, ending inside a split, and empty past a short context; the last split
    of an item to finish merges them.  fp32 sums of up to 1536 terms: 1e-5 of the largest logit is some 80 ulps."""
    say("fp32 key splits", hd)
    shape = synth.ModelShape(2, 256, 256 // hd, 256 // hd, 512, 1008, "fp32")
    draft = synth.ModelShape(1, 128, 128 // hd, 128 // hd, 256, 1008, "fp32")
    prompts = synth.prompts(3, [1510, 700, 3], shape.vocab)
    _compare(shape, draft, prompts, 5, bound=1e-5, prefill_rows=512)
