"""What the library launches, recorded by a HIP runtime that runs nothing
(tests/native/hip_recorder.cpp), in a process of its own without torch."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2510_11331_amd", "libsd.so")

pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="libsd.so not built (run __graft_entry__.build())"),
              pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")]

PRELUDE = '''
import ctypes as C, importlib.util, sys, types
sys.modules["torch"] = types.ModuleType("torch")          # the library is loaded without a HIP runtime of torch's
sys.path.insert(0, sys.argv[2])
R = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
spec = importlib.util.spec_from_file_location("_lib", sys.argv[2] + "/paper_2510_11331_amd/_lib.py")
_lib = importlib.util.module_from_spec(spec); spec.loader.exec_module(_lib)
import synth
L = _lib.lib()

def launches():
    out = []
    for i in range(R.recorder_count()):
        name, v = C.create_string_buffer(512), (C.c_int * 5)()
        R.recorder_get(i, name, 512, v)
        out.append((name.value.decode(),) + tuple(v))        # name, device, workgroups, threads, dynamic LDS, its limit
    R.recorder_clear()
    return out

def cfg(t, d, batch, gamma, prefill_rows, max_ctx=512):
    m = lambda s: _lib.ModelCfg(s.n_layers, s.d_model, s.n_heads, s.n_kv_heads, s.head_dim, s.d_ffn, s.vocab,
                                _lib.SD_DTYPE_BF16 if s.dtype == "bf16" else _lib.SD_DTYPE_F32, s.rope_theta, s.rms_eps)
    c = _lib.Config(m(t), m(d), batch, batch, gamma, max_ctx, 16, batch * max_ctx // 16, batch * max_ctx // 16,
                    prefill_rows, 1.0, 0, 1 << 32, 1 << 33, 1 << 34)
    c.workspace_bytes = L.sd_workspace_bytes(C.byref(c))
    assert c.workspace_bytes
    return c

def context(c):
    keep = []
    def weights(n):
        a = [(C.c_void_p * n)(*[256 * (k + 1) for k in range(n)]) for _ in range(6)]
        keep.append(a)
        return _lib.Weights(256, 256, 256, *[C.cast(x, C.POINTER(C.c_void_p)) for x in a])
    h = C.c_void_p()
    w = weights(c.target.n_layers), weights(c.draft.n_layers)
    _lib.check(L.sd_init(C.byref(c), C.byref(w[0]), C.byref(w[1]), C.byref(h)), "sd_init")
    return h

def prefill(h, lens):
    B, I = len(lens), C.c_int32
    toks = (I * sum(lens))()
    _lib.check(L.sd_prefill(h, B, (I * B)(*range(B)), toks, (I * B)(*lens), (I * B)(*[8] * B), None), "sd_prefill")

def draft_and_verify(h, B, gamma):
    p = 1 << 35
    for i in range(gamma):
        _lib.check(L.sd_draft_step(h, B, p, gamma, i, p, p, p, None), "sd_draft_step")
    _lib.check(L.sd_verify(h, B, p, gamma, p, p, None, None), "sd_verify")
'''


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = tmp_path_factory.mktemp("hip") / "librecorder.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "native", "hip_recorder.cpp"),
                    "-o", str(so)], check=True, capture_output=True, timeout=300)
    return str(so)


def _run(recorder, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, recorder, ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_lds_limit_is_set_on_every_device(recorder):
    """Launches of 64 KB of dynamic LDS and more: the limit is an attribute of the kernel on one device, so a context on
    a second device needs it set there too, also where another context ran the same kernels before."""
    out = _run(recorder, '''
big = set()
for dtype in ("bf16", "fp32"):
    t = synth.ModelShape(2, 1024, 8, 2, 2816, 1008, dtype)
    d = synth.ModelShape(1, 512, 8, 8, 512, 1008, dtype)
    for dev in (0, 1, 0, 2):
        R.recorder_device(dev)
        h = context(cfg(t, d, 64, 8, 1024))
        prefill(h, [130 + k for k in range(4)])
        draft_and_verify(h, 64, 8)
        for name, on, _, _, lds, limit in launches():
            assert on == dev
            if lds >= 64 * 1024:
                assert limit >= lds, (name, dev, lds, limit)
                big.add((name, dev))
        L.sd_destroy(h)
print(len(big))
''')
    assert int(out) >= 12


def test_launches_follow_the_plan(recorder):
    """sd_plan_projection against the projections that prefill, draft and verify launch."""
    out = _run(recorder, '''
import re
n = 0
for t, d, B, gamma, lens in ((synth.MODELS["small_target"], synth.MODELS["small_draft"], 8, 4, [200] * 8),
                             (synth.MODELS["7b_target"].replace(n_layers=2), synth.MODELS["7b_draft"], 1, 4, [129]),
                             (synth.MODELS["13b_target"].replace(n_layers=2), synth.MODELS["13b_draft"], 64, 4, [40] * 64),
                             (synth.ModelShape(2, 320, 5, 5, 2752, 1008, "bf16"), synth.ModelShape(1, 192, 3, 1, 64, 1008, "bf16"), 33, 7, [9] * 33)):
    c = cfg(t, d, B, gamma, 1000)
    h = context(c)
    rows = sum(x - 1 for x in lens)
    chunks = [min(1000, rows - k) for k in range(0, rows, 1000)]
    def expect(ps, M, lm=0):
        m = c.target if ps in (_lib.SD_PASS_VERIFY, _lib.SD_PASS_PREFILL) else c.draft
        seq = []
        for l in range(m.n_layers):
            last = ps >= _lib.SD_PASS_PREFILL and l + 1 == m.n_layers
            seq += [(_lib.SD_PROJ_KV, M)] if last else [(j, M) for j in (_lib.SD_PROJ_QKV, _lib.SD_PROJ_O, _lib.SD_PROJ_GATEUP, _lib.SD_PROJ_DOWN)]
        if lm:
            seq.append((_lib.SD_PROJ_LM_HEAD, lm))
        res = []
        for j, r in seq:
            p = _lib.ProjPlan()
            _lib.check(L.sd_plan_projection(C.byref(c), ps, j, r, C.byref(p)), "sd_plan_projection")
            epi = {0: 3, 1: 3, 2: 1, 3: 2, 4: 1, 5: 0}[j]
            epi = 4 if p.ksplit > 1 else epi
            if p.tile >= 0:
                res.append((f"gemm_rows_kernelINS_7RowTileI" + "".join(f"Li{v}E" for v in (p.mf, p.nf, p.wm, p.wn, p.ks, p.nb)) + f"EELi{epi}E", p.grid, 64 * p.wm * p.wn))
            else:
                res.append((f"gemm_kernelIDF16_Li{p.mt}ELi{p.nt}ELi2ELi{epi}E", p.grid, 64 * p.kw))
        return res
    want = []
    for M in chunks:
        want += expect(_lib.SD_PASS_PREFILL, M) + expect(_lib.SD_PASS_PREFILL_DRAFT, M)
    for i in range(gamma):
        want += expect(_lib.SD_PASS_DRAFT, B * (2 if i == 0 else 1), B)
    want += expect(_lib.SD_PASS_VERIFY, B * (gamma + 1), B * (gamma + 1))
    launches()
    prefill(h, lens)
    draft_and_verify(h, B, gamma)
    got = [x for x in launches() if "gemm_" in x[0]]
    assert len(got) == len(want), (len(got), len(want))
    for g, w in zip(got, want):
        assert w[0] in g[0] and g[2:4] == w[1:], (g, w)
        n += 1
    L.sd_destroy(h)
print(n)
''')
    assert int(out) > 100
