"""Attention of 16-bit caches: the query-tile and key-group arrangements of the
decode kernel, against the oracle."""
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


def _compare(shape, dshape, prompts, gamma, **kw):
    B = len(prompts)
    tw, dw = synth.model_weights(shape, 5), synth.model_weights(dshape, 6)
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
            assert err < BOUND, (k, j, err)


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
