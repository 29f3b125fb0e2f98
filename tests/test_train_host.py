"""CPU tests of the group-wise training attention's entry points: exported as declared, struct layout, host-side validation."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2410_05589_amd import binding as B
from paper_2410_05589_amd import train as TR

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2410_05589_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


def _code():
    return re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "ps_train.h")).read(), flags=re.S)


def test_declared_symbols_and_struct_layout(lib):
    declared = sorted(set(re.findall(r"\bPS_API\s+[a-z_]+\s+(ps_[a-z_]+)\s*\(", _code())))
    assert declared == sorted(TR.EXPORTED_SYMBOLS)
    for n in declared:
        assert getattr(lib, n) is not None
    body = _code()
    body = body[body.index("typedef struct ps_group_attn_args {"):body.index("} ps_group_attn_args;")]
    names = [n for line in re.findall(r"[^;{]+;", body) for n in re.findall(r"\*?\s*([a-z_]+)\s*[,;]", line)]
    assert names == [f[0] for f in TR.ps_group_attn_args._fields_]


def test_validation_on_the_host(lib):
    def args(**kw):
        a = TR.make_args(1, 64, 4, 8, 8, 64, "bf16", 10000.0)
        for n in ("q", "k_", "v", "out", "workspace"):
            setattr(a, n, 0x100000)
        a.workspace_bytes = 1 << 40
        for k_, v in kw.items():
            setattr(a, k_, v)
        return a
    assert TR.ps_group_attention_workspace_bytes(args()) > 0
    assert TR.ps_group_attention(None, None) == B.PS_ERR_NULL
    for kw in (dict(seqs=0), dict(tokens=0), dict(k=-1), dict(n_kv_heads=3), dict(dtype=5), dict(rope_base=0.0)):
        assert TR.ps_group_attention(args(**kw), None) == B.PS_ERR_SHAPE, kw
        assert TR.ps_group_attention_workspace_bytes(args(**kw)) == 0
    for kw in (dict(head_dim=96), dict(k=16), dict(tokens=1 << 20), dict(k=15, n_heads=32768, n_kv_heads=32768, head_dim=128)):
        assert TR.ps_group_attention(args(**kw), None) == B.PS_ERR_UNSUPPORTED, kw
    for n in ("q", "k_", "v", "out", "workspace"):
        assert TR.ps_group_attention(args(**{n: None}), None) == B.PS_ERR_NULL, n
    need = TR.ps_group_attention_workspace_bytes(args())
    assert TR.ps_group_attention(args(workspace_bytes=need - 1), None) == B.PS_ERR_WORKSPACE
    assert TR.ps_group_attention(args(workspace=0x100010), None) == B.PS_ERR_WORKSPACE


def test_launches_stay_within_the_limits_of_a_launch(lib):
    """Work items of a launch in x are at most 2^32 - 1 and workgroups in y and z at most 65535 each, whatever the
    sizes that the entry point takes; and the attention's workgroups cover all rows of all heads and sequences."""
    from paper_2410_05589_amd import debug as DBG
    rows_of, seen = {0: 64, 2: 128, 3: 32, 4: 32}, set()     # (1, the bf16 tiles of whole groups, counts otherwise)
    for dtype, seqs, T, k, nq, nkv, d in [
            ("bf16", 1, 2048, 4, 32, 32, 128), ("bf16", 4096, 1, 0, 4096, 1, 64), ("bf16", 4097, 1, 0, 4096, 1, 64),
            ("bf16", 65535, 1, 0, 8192, 1, 64), ("bf16", 1, (1 << 20) - 15, 15, 128, 8, 128), ("bf16", 65535, 4, 3, 640, 1, 128),
            ("f32", 2, 300, 3, 8, 8, 64), ("f32", 1, 1024, 15, 32768, 1, 64), ("f32", 1, (1 << 20) - 15, 15, 32, 8, 128),
            ("f32", 65535, 1, 0, 65535, 1, 64), ("f32", 3, 1 << 19, 0, 1024, 1, 64),
            ("f32", 1, (1 << 20) - 15, 15, 8190, 1, 64), ("f32", 1, (1 << 20) - 15, 15, 8190, 1, 128)]:
        a = TR.make_args(seqs, T, k, nq, nkv, d, dtype, 10000.0)
        st, g = DBG.ps_train_debug_launch(a)
        tag = (dtype, seqs, T, k, nq, g)
        assert st == B.PS_OK, tag
        for (x, y, z), threads in ((g["grid"], g["threads"]), (g["rope_grid"] + (1,), g["rope_threads"])):
            assert x * threads < 1 << 32 and 1 <= y <= 65535 and 1 <= z <= 65535, tag
        assert g["rope_grid"][0] == T + k, tag
        if g["kernel"] in rows_of:
            blocks = -(-T * (k + 1) // rows_of[g["kernel"]]) * nq * (seqs if dtype == "bf16" else 1)
            x, y, z = g["grid"]
            assert blocks <= x * y < blocks + x and blocks < 1 << 32 and z == (1 if dtype == "bf16" else seqs), tag
        seen.add(g["kernel"])
    assert seen >= set(rows_of), seen
    huge = TR.make_args(1, 1 << 19, 15, 32768, 1, 64, "f32", 10000.0)           # 2^33 blocks of 32 rows
    assert DBG.ps_train_debug_launch(huge)[0] == B.PS_ERR_UNSUPPORTED and TR.ps_group_attention_workspace_bytes(huge) == 0
    assert DBG.ps_train_debug_launch(TR.make_args(1, 64, 16, 8, 8, 64, "bf16", 10000.0))[0] == B.PS_ERR_UNSUPPORTED
    assert DBG.ps_train_debug_launch(TR.make_args(0, 64, 4, 8, 8, 64, "bf16", 10000.0))[0] == B.PS_ERR_SHAPE


def test_which_float32_calls_are_short(lib):
    """Both sides of the line: 704 workgroups of 32 rows (head_dim 64), 400 (128); blocks of 32 rows cover the rows."""
    from paper_2410_05589_amd import debug as DBG
    for d, want, calls in ((64, 4, [(1, 1, 0, 1), (1, 700, 3, 8), (11, 256, 0, 8)]), (64, 3, [(1, 705, 3, 8), (11, 257, 0, 8)]),
                           (128, 4, [(1, 400, 3, 8), (1, 12800, 0, 1)]), (128, 0, [(1, 401, 3, 8), (1, 12801, 0, 1)])):
        for seqs, T, k, nq in calls:
            st, g = DBG.ps_train_debug_launch(TR.make_args(seqs, T, k, nq, nq, d, "f32", 10000.0))
            assert st == B.PS_OK and g["kernel"] == want, (d, seqs, T, k, nq, g)
            x, y, z = g["grid"]
            assert z == seqs and x * y == -(-T * (k + 1) // (64 if want == 0 else 32)) * nq, (d, seqs, T, k, nq, g)
            assert g["threads"] == {4: 512, 3: 256, 0: 512}[want]


def test_which_calls_take_the_16_row_kernel(lib):
    """Both sides of every limit of the rule: T 32, k 4, group sizes that divide 32, 256 workgroups, 8192 key rows."""
    from paper_2410_05589_amd import debug as DBG
    for want, calls in ((1, [(1, 32, 4, 8, 8), (1, 32, 8, 32, 8), (1, 1, 7, 8, 8), (1, 1, 15, 8, 8), (1, 16, 14, 8, 8), (1, 25, 8, 36, 36)]),
                        (2, [(1, 33, 4, 8, 8), (1, 32, 3, 8, 8), (1, 32, 7, 8, 8), (1, 32, 15, 8, 8), (1, 32, 8, 33, 11), (1, 26, 8, 36, 36),
                             (1, 16, 10, 48, 48), (8, 32, 8, 40, 40)])):
        for seqs, T, k, nq, nkv in calls:
            for d in (64, 128):
                st, g = DBG.ps_train_debug_launch(TR.make_args(seqs, T, k, nq, nkv, d, "bf16", 10000.0))
                assert st == B.PS_OK and g["kernel"] == want, (seqs, T, k, nq, nkv, g)


def test_plans_of_the_largest_calls_do_not_overflow(tmp_path):
    """The host code that plans a call, built with checks for signed overflow, on the most heads, sequences
    and tokens that the entry points take."""
    from paper_2410_05589_amd import build
    inc = ["-I", os.path.join(ROOT, "include"), "-I", build.CSRC]
    obj, main, exe = (str(tmp_path / n) for n in ("train.o", "main.cpp", "main"))

    def run(cmd):
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert res.returncode == 0, (cmd, res.stdout[-2000:])
        return res.stdout
    checks = [a for f in ("-fsanitize=signed-integer-overflow", "-fno-sanitize-recover=signed-integer-overflow") for a in ("-Xarch_host", f)]
    run([build.hipcc_path(), "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", *checks, *inc, "-c", "-o", obj,
         os.path.join(build.CSRC, "ps_train.hip")])
    image = re.search(r"U (__hip_fatbin\w*)", run(["nm", obj])).group(1)        # (no device code in this build)
    calls = [(dt, 65535, 1, 0, 65535, nkv, 64) for dt in ("bf16", "f32") for nkv in (1, 65535)]
    calls += [("bf16", 65535, (1 << 20) - 15, 15, 65534, 32767, 64), ("f32", 1, (1 << 20) - 15, 15, 8190, 1, 128)]
    rows = ",".join("{%s, %d, %d, %d, %d, %d, %d}" % ("PS_BF16" if c[0] == "bf16" else "PS_F32", *c[1:]) for c in calls)
    open(main, "w").write("""#include <cstdio>
#include "ps_train.h"
#include "ps_draft_debug.h"
extern "C" { extern const char %s[4096] = {}; }
int main() {
    const int calls[][7] = {%s};
    for (auto& c : calls) {
        ps_group_attn_args a = {};
        a.dtype = c[0]; a.seqs = c[1]; a.tokens = c[2]; a.k = c[3]; a.n_heads = c[4]; a.n_kv_heads = c[5]; a.head_dim = c[6]; a.rope_base = 10000.f;
        unsigned out[8];
        if (ps_train_debug_launch(&a, out) != PS_OK || ps_group_attention_workspace_bytes(&a) == 0) return printf("refused: %%d %%d\\n", a.seqs, a.n_heads), 3;
    }
    return 0;
}
""" % (image, rows))
    run([build.hipcc_path(), "-x", "c++", "-std=c++17", *inc, "-c", "-o", main + ".o", main])
    run([build.hipcc_path(), *checks[:2], "-o", exe, main + ".o", obj])
    run([exe])
