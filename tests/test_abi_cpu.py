"""C ABI checks that need no GPU: libsd loads, exports every function
include/sd.h declares, sizes follow the documented layouts, and invalid
arguments are rejected on the host before anything is enqueued."""
import ctypes as C
import os
import re

import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_11331_amd", "libsd.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libsd.so not built (run __graft_entry__.build())")


def header_functions():
    names = set()
    for h in ("sd.h", "sd_sched.h"):
        src = open(os.path.join(ROOT, "include", h)).read()
        src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
        names |= set(re.findall(r"\b(sd_[a-z_]+)\s*\(", src))
    return sorted(names)


def test_exports_every_declared_function():
    from paper_2510_11331_amd import _lib
    L = _lib.lib()
    names = header_functions()
    assert len(names) >= 15
    for n in names:
        assert hasattr(L, n), n
    assert set(names) == set(_lib.EXPORTS)


def make_cfg(tshape=None, dshape=None, **kw):
    from paper_2510_11331_amd import _lib
    from paper_2510_11331_amd.engine import model_cfg
    c = _lib.Config()
    c.target = model_cfg(tshape or synth.MODELS["tiny_target"])
    c.draft = model_cfg(dshape or synth.MODELS["tiny_draft"])
    c.max_slots, c.max_batch, c.gamma_max, c.max_ctx = 4, 2, 4, 128
    c.kv_block, c.kv_blocks_target, c.kv_blocks_draft = 16, 32, 32
    c.prefill_rows, c.temperature, c.greedy = 64, 1.0, 0
    for k, v in kw.items():
        setattr(c, k, v)
    return c


def test_sizes_and_validation():
    from paper_2510_11331_amd import _lib
    L = _lib.lib()
    c = make_cfg()
    t = synth.MODELS["tiny_target"]
    # pool: per layer [kv heads][blocks][K|V][16 tokens x head_dim] in the model dtype (fp32 here)
    assert L.sd_kv_pool_bytes(C.byref(c), 0) == t.n_layers * 32 * 2 * t.n_kv_heads * 16 * t.head_dim * 4
    assert L.sd_workspace_bytes(C.byref(c)) > 0
    bad = [dict(kv_block=8), dict(gamma_max=0), dict(gamma_max=17), dict(max_batch=5),
           dict(temperature=0.0), dict(prefill_rows=0), dict(max_ctx=1), dict(max_ctx=32769)]
    for kw in bad:
        cb = make_cfg(**kw)
        assert L.sd_workspace_bytes(C.byref(cb)) == 0, kw
        h = C.c_void_p()
        w = _lib.Weights()
        assert L.sd_init(C.byref(cb), C.byref(w), C.byref(w), C.byref(h)) == _lib.SD_EINVAL
    # shapes the kernels do not cover are refused: head_dim 96, vocab not a multiple of 16
    for shape in (synth.ModelShape(1, 192, 2, 2, 512, 1024, "fp32"),
                  synth.ModelShape(1, 128, 2, 2, 512, 1000, "fp32"),
                  synth.ModelShape(1, 128, 2, 2, 520, 1024, "bf16")):
        assert L.sd_workspace_bytes(C.byref(make_cfg(dshape=shape))) == 0
    # valid configuration but null weights / buffers: rejected before any HIP call
    h = C.c_void_p()
    w = _lib.Weights()
    assert L.sd_init(C.byref(c), C.byref(w), C.byref(w), C.byref(h)) == _lib.SD_EINVAL
    assert L.sd_init(None, None, None, C.byref(h)) == _lib.SD_EINVAL


def test_context_free_and_null_context_errors():
    from paper_2510_11331_amd import _lib
    L = _lib.lib()
    E = _lib.SD_EINVAL
    assert L.sd_accept_resample(0, 4, 16, 0, None, None, None, None, None, None, None) == E
    assert L.sd_accept_resample(1, 0, 16, 0, 1, 1, 1, 1, 1, 1, None) == E
    # rows are read as 16-byte vectors: a vocabulary that is not a multiple of
    # 4, or q / p rows that do not start on 16 bytes, are refused before any
    # launch (the pointers below are never dereferenced)
    A = 1 << 20
    for V in (1, 2, 3, 1001, 31999, 32002):
        assert L.sd_accept_resample(2, 4, V, 0, A, A, A, A, A, A, None) == E, V
    assert L.sd_accept_resample(2, 4, 1024, 0, A, A + 8, A, A, A, A, None) == E
    assert L.sd_accept_resample(2, 4, 1024, 0, A, A, A + 4, A, A, A, None) == E
    assert L.sd_accept_resample(2, 4, 32772, 0, A, A, A, A, A, A, None) == E
    assert L.sd_draft_step(None, 1, 1, 4, 0, 1, 1, 1, None) == E
    assert L.sd_verify(None, 1, 1, 4, 1, 1, None, None) == E
    assert L.sd_kv_commit(None, 1, 1, 4, 1, 1, None) == E
    assert L.sd_release(None, 0) == E
    assert L.sd_profile(None, 1) == E
    for code in (0, -1, -2, -3, -4):
        assert len(_lib.strerror(code)) >= 2 and _lib.strerror(code) != str(code)


def test_plan_projection():
    """The plan query: shapes and passes of a configuration, refusals, and plans that cover their outputs."""
    from paper_2510_11331_amd import _lib
    L = _lib.lib()
    p = _lib.ProjPlan()
    plan = lambda c, ps, pj, rows: L.sd_plan_projection(C.byref(c), ps, pj, rows, C.byref(p))
    t, d = synth.MODELS["small_target"], synth.MODELS["small_draft"]
    c = make_cfg(t, d, prefill_rows=700)
    widths = {_lib.SD_PROJ_QKV: lambda m: ((m.n_heads + 2 * m.n_kv_heads) * m.head_dim, m.d_model),
              _lib.SD_PROJ_KV: lambda m: (2 * m.n_kv_heads * m.head_dim, m.d_model),
              _lib.SD_PROJ_O: lambda m: (m.d_model, m.d_model), _lib.SD_PROJ_GATEUP: lambda m: (2 * m.d_ffn, m.d_model),
              _lib.SD_PROJ_DOWN: lambda m: (m.d_model, m.d_ffn), _lib.SD_PROJ_LM_HEAD: lambda m: (m.vocab, m.d_model)}
    for ps, m in ((_lib.SD_PASS_VERIFY, t), (_lib.SD_PASS_DRAFT, d), (_lib.SD_PASS_PREFILL, t), (_lib.SD_PASS_PREFILL_DRAFT, d)):
        refused = _lib.SD_PROJ_LM_HEAD if ps >= _lib.SD_PASS_PREFILL else _lib.SD_PROJ_KV
        for pj, nk in widths.items():
            for rows in (1, 10, 64) + ((65, 256, 700) if ps != _lib.SD_PASS_DRAFT else ()):
                rc = plan(c, ps, pj, rows)
                assert rc == (_lib.SD_EINVAL if pj == refused else _lib.SD_OK), (ps, pj, rows)
                if rc != _lib.SD_OK:
                    continue
                assert (p.M, (p.N, p.K)) == (rows, nk(m)) and 1 <= p.ksplit <= 6
                if p.tile >= 0:
                    bm, bn = 16 * p.mf * p.wm, 16 * p.nf * p.wn
                    assert p.grid == -(-p.N // bn) * -(-rows // bm) * p.ksplit
                else:
                    assert p.tile_unit or p.grid * 16 * p.nt >= p.N * p.ksplit * -(-rows // (16 * p.mt))
        assert plan(c, ps, _lib.SD_PROJ_QKV, 0) == _lib.SD_EINVAL
        assert plan(c, ps, _lib.SD_PROJ_QKV, 705) == _lib.SD_EINVAL     # the workspace holds 704 (64 drafting) rows
    assert plan(c, 4, 0, 1) == plan(c, 0, 6, 1) == plan(c, -1, 0, 1) == plan(c, 0, -1, 1) == _lib.SD_EINVAL
    assert plan(make_cfg(prefill_rows=0), 0, 0, 1) == _lib.SD_EINVAL
    f32 = make_cfg()
    assert plan(f32, _lib.SD_PASS_PREFILL, _lib.SD_PROJ_GATEUP, 64) == _lib.SD_OK and p.tile == -1
