"""CPU tests of the C-ABI library: it loads, exports what the header declares, and its
host-side validation reports errors before touching any device."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2410_05589_amd import binding as B
from paper_2410_05589_amd import debug as DBG
from paper_2410_05589_amd.configs import WORKLOADS, small_shape

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2410_05589_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


def _declared_functions(header):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\bPS_API\s+[a-z_ ]+\*?\s+(ps_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    declared = _declared_functions("ps_draft.h")
    assert sorted(B.EXPORTED_SYMBOLS) == declared
    for name in declared:
        assert getattr(lib, name) is not None
    debug = _declared_functions("ps_draft_debug.h")
    assert sorted(DBG.EXPORTED_SYMBOLS) == debug
    for name in debug:
        assert getattr(lib, name) is not None


def test_nothing_else_is_exported(lib):
    """The dynamic symbol table holds exactly the ps_* functions the headers declare."""
    import subprocess
    out = subprocess.run(["nm", "-D", "--defined-only", B.LIB_PATH], stdout=subprocess.PIPE, text=True, check=True).stdout
    exported = sorted(l.split()[-1] for l in out.splitlines() if l.split()[-1].startswith("ps_"))
    declared = sorted(sum((_declared_functions(h) for h in ("ps_draft.h", "ps_verify.h", "ps_draft_debug.h", "ps_train.h")), []))
    assert exported == declared


def test_struct_layouts_match_header():
    # field order of the ctypes mirrors follows the header text
    text = open(os.path.join(ROOT, "include", "ps_draft.h")).read()
    body = text[text.index("typedef struct ps_draft_config {"):text.index("} ps_draft_config;")]
    names = re.findall(r"\b(?:int32_t|float|uint32_t)\s+([a-z_]+);", body)
    assert names == [f[0] for f in B.ps_draft_config._fields_]
    body = text[text.index("typedef struct ps_draft_weights {"):text.index("} ps_draft_weights;")]
    assert re.findall(r"const void\*\s+([a-z_]+);", body) == list(B.WEIGHT_NAMES + B.INPUT_WEIGHT_NAMES)
    body = text[text.index("typedef struct ps_draft_step_args {"):text.index("} ps_draft_step_args;")]
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    names = [n for line in re.findall(r"[^;{]+;", body) for n in re.findall(r"\*?\s*\**([a-z_]+)\s*[,;]", line)]
    assert names == [f[0] for f in B.ps_draft_step_args._fields_]
    assert ctypes.sizeof(B.ps_draft_config) == 15 * 4


def _cfg(name="c1", **kw):
    wl = WORKLOADS[name]
    c = B.make_config(wl.shape, max_batch=1, max_new=6, max_positions=2048, max_topk=8)
    for k, v in kw.items():
        setattr(c, k, v)
    return c


def test_workspace_bytes_for_the_five_workloads(lib):
    for name, wl in WORKLOADS.items():
        c = B.make_config(wl.shape, max_batch=wl.batch, max_new=max(wl.n_new_mix or (wl.n_new,)),
                          max_positions=4200, max_topk=8, k_max=wl.k)
        n = B.ps_draft_workspace_bytes(c)
        assert n > 0 and n % 256 == 0, name
        assert n < 2 << 30


def test_config_validation(lib):
    assert B.ps_draft_workspace_bytes(_cfg()) > 0
    bad = [dict(hidden=0), dict(n_kv_heads=3), dict(dtype=7), dict(max_batch=0), dict(k_max=-1),
           dict(rope_base=0.0), dict(flags=8), dict(max_positions=3), dict(max_topk=0), dict(rms_eps=-1.0)]
    for kw in bad:
        c = _cfg(**kw)
        assert B.ps_draft_workspace_bytes(c) == 0, kw
        w = B.ps_draft_weights()
        for n in B.WEIGHT_NAMES:
            setattr(w, n, 0x1000)
        st, h = B.ps_draft_init(c, w, 0x100000, 1 << 40, None)
        assert st == B.PS_ERR_CONFIG, kw
    unsupported = [dict(head_dim=96, n_heads=32, n_kv_heads=32), dict(hidden=4100), dict(ffn=11012),
                   dict(max_batch=32), dict(max_topk=33)]
    for kw in unsupported:
        c = _cfg(**kw)
        w = B.ps_draft_weights()
        for n in B.WEIGHT_NAMES:
            setattr(w, n, 0x1000)
        st, h = B.ps_draft_init(c, w, 0x100000, 1 << 40, None)
        assert st == B.PS_ERR_UNSUPPORTED, kw


def test_exchange_buffers_the_kernels_cannot_address_are_refused(lib):
    """The kernels use 32-bit byte offsets into every exchange buffer: a legal configuration whose attention
    partials (or any other exchange buffer) would reach 4 GiB is unsupported, not silently wrapped."""
    ok = _cfg(max_batch=4, max_positions=1 << 15)
    assert B.ps_draft_workspace_bytes(ok) > 0
    for kw in (dict(max_batch=4, max_positions=1 << 20), dict(max_positions=(1 << 24) + 1)):
        c = _cfg(**kw)
        assert B.ps_draft_workspace_bytes(c) == 0, kw
        w = B.ps_draft_weights()
        for n in B.WEIGHT_NAMES:
            setattr(w, n, 0x1000)
        assert B.ps_draft_init(c, w, 0x100000, 1 << 44, None)[0] == B.PS_ERR_UNSUPPORTED, kw
        assert DBG.ps_draft_debug_plan(c, 1, 1, 5, 0, 256, 160 * 1024)[0] == B.PS_ERR_UNSUPPORTED, kw


def test_init_null_and_workspace_errors(lib):
    c = _cfg()
    w = B.ps_draft_weights()
    for n in B.WEIGHT_NAMES:
        setattr(w, n, 0x1000)
    need = B.ps_draft_workspace_bytes(c)
    assert B.ps_draft_init(None, w, 0x100000, need, None)[0] == B.PS_ERR_NULL
    assert B.ps_draft_init(c, None, 0x100000, need, None)[0] == B.PS_ERR_NULL
    assert B.ps_draft_init(c, w, None, need, None)[0] == B.PS_ERR_NULL
    assert B.ps_draft_init(c, w, 0x100000, need - 1, None)[0] == B.PS_ERR_WORKSPACE
    assert B.ps_draft_init(c, w, 0x100010, need, None)[0] == B.PS_ERR_WORKSPACE
    w2 = B.ps_draft_weights()
    for n in B.WEIGHT_NAMES:
        setattr(w2, n, 0x1000)
    w2.w_lm = None
    assert B.ps_draft_init(c, w2, 0x100000, need, None)[0] == B.PS_ERR_NULL
    # g_final may be NULL only without the final norm
    w3 = B.ps_draft_weights()
    for n in B.WEIGHT_NAMES:
        setattr(w3, n, 0x1000)
    w3.g_final = None
    assert B.ps_draft_init(c, w3, 0x100000, need, None)[0] == B.PS_ERR_NULL


def test_step_and_free_with_null_context(lib):
    a = B.ps_draft_step_args()
    assert B.ps_draft_step(None, a, None) == B.PS_ERR_NULL
    assert B.ps_draft_last_status(None, None) == B.PS_ERR_NULL
    assert DBG.ps_draft_debug_spin_limit(None, 1) == B.PS_ERR_NULL
    assert DBG.ps_measure_stream_read(None, 1024, None) == B.PS_ERR_NULL
    assert DBG.ps_measure_stream_read(0x1000, 1000, None) == B.PS_ERR_SHAPE
    assert DBG.ps_measure_copy(0x1000, 0x2000, 8, None) == B.PS_ERR_SHAPE
    B.ps_draft_free(None)


def test_strerror(lib):
    seen = set()
    for st in range(0, -10, -1):
        s = B.ps_draft_strerror(st)
        assert s and s != "unknown status"
        seen.add(s)
    assert len(seen) == 10
    assert B.ps_draft_strerror(-99) == "unknown status"


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "LIB_PATH", "/nonexistent/libps_draft.so")
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        B.load_library()


PS_U, PS_WAVES = 8, 8


def _plan(lib, cfg, batch, n_new, k, n_cu=256, lds=160 * 1024, all_rows=0):
    st, plans = DBG.ps_draft_debug_plan(cfg, batch, n_new, k, all_rows, n_cu, lds)
    return (st, plans) if st == B.PS_OK else (st, None)


def _check_plan(cfg, plans, batch, n_new, k, n_cu, lds):
    """What the device code relies on (it has no bounds checks of its own for these)."""
    esz_step = 32 if cfg.dtype == B.PS_BF16 else 16          # elements per 64-byte step
    for ph, d in enumerate(plans):
        tag = (ph, d, batch, n_new, k, n_cu, lds)
        S, KW = 1 << d["s_log"], 1 << d["kw_log"]
        assert d["Kt"] % PS_U == 0 and d["Kt"] * esz_step >= d["K"] > (d["Kt"] - PS_U) * esz_step, tag
        assert 1 <= KW <= PS_WAVES and 1 <= S <= 8, tag
        if ph == 4:
            assert S == 1, tag                                 # the LM head keeps a row's logits in one workgroup
            assert min(n_cu, d["T"]) <= 512, tag               # one thread per workgroup in the final merge
        assert d["Gs"] == n_cu >> d["s_log"] and d["Gs"] >= 1, tag
        assert d["per_round"] == d["Gs"] * (PS_WAVES >> d["kw_log"]), tag
        assert d["rounds"] == -(-d["T"] // d["per_round"]), tag    # every tile is taken exactly once
        ng = d["Kt"] // PS_U
        sizes = [((ng * (s + 1)) >> d["s_log"]) - ((ng * s) >> d["s_log"]) for s in range(S)]
        pg, npc = d["piece_groups"], d["npieces"]
        assert min(sizes) >= 1 and pg >= KW, tag
        for sz in sizes:
            assert -(-sz // pg) == npc, tag                    # the slices walk through their pieces in step
            assert sz - (npc - 1) * pg >= KW, tag              # every piece gives each wavefront of a tile a group
        assert d["lds_bytes"] <= lds, tag
        arrays = 2 if cfg.dtype == B.PS_BF16 else 1
        assert d["lds_bytes"] >= d["rows"] * arrays * pg * PS_U * 64, tag   # the piece of the panel fits
        # the panel: behind what every phase keeps at the start of LDS and, where wavefronts share a tile, their partial sums; in units
        # at multiples of 256 bytes (their addresses are exchanged below that), and the tiles' logits behind it
        mt = -(-batch * (n_new + k) // 16)
        assert d["panel_off"] >= 1024 + 2304 + (PS_WAVES * mt * 1024 if KW > 1 else 0), tag
        if d["units"]:
            assert d["rows"] > 16 and d["panel_off"] % 256 == 0 and d["rs"] % 256 == 0 and d["rs"] >= -(-d["rows"] // 16) * 256, tag
        else:
            assert d["rs"] >= pg * PS_U * 64, tag
        part = pg * PS_U * 4 * d["rs"] if d["units"] else d["rows"] * d["rs"]
        logits = d["rounds"] * (PS_WAVES // KW) * d["rows"] * 64 if ph == 4 else 0
        assert d["panel_off"] + arrays * part + logits <= d["lds_bytes"], tag
        assert 6 <= d["g2_log"] <= 9, tag                        # whole wavefronts of the 512 threads along a row
        if d["ahead"]:                                           # a thread's share of a piece: one group of at most 8 rows
            assert ph == 4 and npc > 1 and pg * PS_U * 4 <= 1 << d["g2_log"] and d["rows"] <= (512 >> d["g2_log"]) * 8, tag
        assert d["by_piece"] == (ph == 4 and npc > 1 and d["rounds"] > 1 and KW == 1), tag   # (sums wait where one wavefront's logits go)


def test_phase_plans_of_the_five_workloads(lib):
    for name, wl in WORKLOADS.items():
        n_max = max(wl.n_new_mix) if wl.n_new_mix else wl.n_new
        cfg = B.make_config(wl.shape, max_batch=wl.batch, max_new=n_max, max_positions=8192, max_topk=wl.topk, k_max=wl.k)
        for n_new in (sorted(set(wl.n_new_mix)) if wl.n_new_mix else [wl.n_new]):
            st, plans = _plan(lib, cfg, wl.batch, n_new, wl.k)
            assert st == B.PS_OK, (name, n_new)
            _check_plan(cfg, plans, wl.batch, n_new, wl.k, 256, 160 * 1024)


def test_attention_plans_of_the_bf16_workloads_and_of_a_sweep(lib):
    """The bf16 attention's blocks (host logic of ps_draft_step): the block sizes the timed workloads were measured
    fastest with; and for random batches on several device sizes what the device code relies on: the blocks cover
    every sequence, merge items exist exactly when some sequence spans several blocks, and a block size is only
    raised while that spares the workgroups a round of units or the merge."""
    import random
    from paper_2410_05589_amd import inputs
    expect = {"c1": (4, 32, 0), "c2": (2, 160, 40), "c4": (4, 192, 40)}
    for name, (nk, units, merges) in expect.items():
        wl = WORKLOADS[name]
        cfg = B.make_config(wl.shape, max_batch=wl.batch, max_new=6, max_positions=8192, max_topk=wl.topk, k_max=wl.k)
        st, ap = DBG.ps_draft_debug_attn_plan(cfg, wl.kv_len, wl.n_new, wl.k, 256)
        assert st == B.PS_OK and (ap["nk"], ap["units"], ap["merge_items"]) == (nk, units, merges), (name, ap)
    wl = WORKLOADS["c3"]
    cfg = B.make_config(wl.shape, max_batch=wl.batch, max_new=1, max_positions=8192, max_topk=wl.topk, k_max=wl.k)
    st, ap = DBG.ps_draft_debug_attn_plan(cfg, inputs.draw_kv_len(wl), wl.n_new, wl.k, 256)
    assert st == B.PS_OK and ap == {"nk": 16, "units": 256, "blocks": 256, "merge_items": 0}, ap
    f32 = B.make_config(WORKLOADS["c0"].shape, max_batch=1, max_new=1, max_positions=128, max_topk=4, k_max=4)
    assert DBG.ps_draft_debug_attn_plan(f32, (64,), 1, 4, 256)[0] == B.PS_ERR_UNSUPPORTED
    rnd = random.Random(11)
    for _ in range(300):
        n_kv = rnd.choice([1, 2, 4, 8])
        grp = rnd.choice([1, 2, 4])
        shape = small_shape("bf16", hidden=n_kv * grp * 64, n_heads=n_kv * grp, n_kv_heads=n_kv, head_dim=64, ffn=1024, vocab=1000)
        n_new, k = rnd.randint(1, 4), rnd.randint(0, 4)
        M = n_new + k
        batch = rnd.randint(1, max(1, min(8, 64 // (grp * M))))
        kv = [rnd.choice([0, 1, 127, 128, 129, rnd.randint(0, 40000)]) for _ in range(batch)]
        cfg = B.make_config(shape, max_batch=batch, max_new=n_new, max_positions=40000 + M, max_topk=8, k_max=max(k, 1))
        n_cu = rnd.choice([256, 304, 80, 7])
        st, ap = DBG.ps_draft_debug_attn_plan(cfg, kv, n_new, k, n_cu)
        assert st == B.PS_OK, (st, kv)
        ch = 128 * ap["nk"]
        assert ap["nk"] in (1, 2, 4, 8, 16)
        nch = [max(1, -(-l // ch)) for l in kv]
        npass = -(-grp * M // 16)
        assert ap["blocks"] == n_kv * sum(nch) and ap["units"] == ap["blocks"] * npass, (ap, kv)
        assert ap["merge_items"] == n_kv * -(-grp * M // 8) * sum(1 for n in nch if n > 1), (ap, kv)
        if ap["nk"] > 1:   # the next smaller size would cost a round of units more, or is the one that needs the merge
            nch2 = [max(1, -(-l // (ch // 2))) for l in kv]
            more_rounds = -(-n_kv * sum(nch2) * npass // n_cu) > -(-ap["units"] // n_cu)
            assert more_rounds or (max(nch2) > 1 and max(nch) == 1) or max(nch2) > 1, (ap, kv)
    assert DBG.ps_draft_debug_attn_plan(cfg, kv, n_new, k, 0)[0] == B.PS_ERR_SHAPE


def test_phase_plans_over_a_sweep_of_shapes_and_devices(lib):
    import random
    rnd = random.Random(7)
    checked = 0
    seen = {"units": 0, "ahead": 0, "by_piece": 0, "ahead, not by piece": 0}
    for _ in range(400):
        dtype = rnd.choice(["bf16", "f32"])
        mul = 32 if dtype == "bf16" else 16
        head_dim = rnd.choice([64, 128])
        n_kv = rnd.choice([1, 2, 4, 8])
        n_heads = n_kv * rnd.choice([1, 2, 4])
        hidden = n_heads * head_dim
        ffn = mul * rnd.randint(1, 500)
        vocab = rnd.randint(16, 200000)
        shape = small_shape(dtype, hidden=hidden, n_heads=n_heads, n_kv_heads=n_kv, head_dim=head_dim, ffn=ffn, vocab=vocab)
        k = rnd.randint(0, 8)
        n_new = rnd.randint(1, 6)
        grp = n_heads // n_kv
        batch = rnd.randint(1, max(1, min(8, 64 // (n_new + k), 64 // (grp * (n_new + k)) if grp * (n_new + k) <= 64 else 1)))
        if grp * (n_new + k) > 64 or batch * (n_new + k) > 64:
            continue
        cfg = B.make_config(shape, max_batch=batch, max_new=n_new, max_positions=4096, max_topk=8, k_max=max(k, 1))
        for n_cu, lds in ((256, 160 * 1024), (256, 64 * 1024), (304, 160 * 1024), (80, 64 * 1024), (7, 96 * 1024)):
            st, plans = _plan(lib, cfg, batch, n_new, k, n_cu=n_cu, lds=lds, all_rows=rnd.randint(0, 1))
            assert st in (B.PS_OK, B.PS_ERR_UNSUPPORTED), (st, hidden, ffn, vocab)
            if st == B.PS_OK:
                _check_plan(cfg, plans, batch, n_new, k, n_cu, lds)
                checked += 1
                lm = plans[4]
                for n in ("units", "ahead", "by_piece"):
                    seen[n] += lm[n]
                seen["ahead, not by piece"] += lm["ahead"] and not lm["by_piece"]
    assert checked > 500 and min(seen.values()) > 20, (checked, seen)


# (dtype, hidden, ffn, heads, kv heads), (batch, n_new, k), phase, slices: both sides of every line of the rule on 256 compute units
SLICES = [
    ("bf16", 4096, 10240, 8, 8, (2, 1, 5), 2, 2), ("bf16", 4096, 10272, 8, 8, (2, 1, 5), 2, 1),      # gate/up: 5/8 of 2048 wavefronts, none, ...
    ("bf16", 4096, 5120, 8, 8, (3, 1, 5), 2, 4), ("bf16", 4096, 5152, 8, 8, (3, 1, 5), 2, 2),        # ... two ...
    ("bf16", 4096, 2560, 8, 8, (4, 1, 5), 2, 8), ("bf16", 4096, 2592, 8, 8, (4, 1, 5), 2, 4),        # ... and four slices
    ("bf16", 8192, 1024, 8, 8, (1, 1, 5), 2, 8), ("bf16", 7168, 2048, 8, 8, (1, 1, 5), 2, 8),
    ("f32", 4096, 6128, 8, 8, (3, 1, 5), 2, 8), ("f32", 4096, 6144, 8, 8, (3, 1, 5), 2, 2),          # 3/4, over all rounds
    ("f32", 4096, 3056, 8, 8, (3, 1, 5), 2, 8), ("f32", 4096, 3072, 8, 8, (3, 1, 5), 2, 4), ("f32", 4096, 4352, 8, 8, (3, 1, 5), 2, 8),
    ("f32", 4096, 2816, 32, 4, (3, 1, 5), 0, 8), ("f32", 4096, 2816, 32, 8, (3, 1, 5), 0, 4),
    ("bf16", 4096, 2816, 8, 4, (3, 1, 5), 0, 8), ("bf16", 4096, 2816, 16, 2, (3, 1, 5), 0, 4),       # QKV: a quarter with K 4096, up to 24 rows
    ("bf16", 4096, 2816, 16, 2, (4, 1, 5), 0, 4), ("bf16", 4096, 2816, 16, 2, (5, 1, 4), 0, 8),
    ("bf16", 4352, 2816, 32, 8, (3, 1, 5), 0, 8), ("bf16", 4352, 2816, 32, 16, (3, 1, 5), 0, 4), ("bf16", 4096, 2816, 32, 8, (8, 1, 3), 0, 8),
    ("bf16", 2048, 2816, 16, 16, (3, 1, 5), 1, 8), ("bf16", 4096, 2816, 16, 4, (3, 1, 5), 1, 8),     # output projection: K 2048, one tile a wavefront or not
    ("bf16", 4352, 2816, 16, 4, (3, 1, 5), 1, 4), ("bf16", 2304, 2816, 18, 18, (3, 1, 5), 1, 4),
    ("bf16", 2048, 2048, 16, 16, (1, 1, 5), 3, 8), ("bf16", 2048, 2304, 16, 16, (1, 1, 5), 3, 4), ("bf16", 4352, 2048, 16, 16, (1, 1, 5), 3, 4)]


@pytest.mark.parametrize("shape,step,phase,slices", [(s[:5], s[5], s[6], s[7]) for s in SLICES])
def test_fewer_slices_only_where_enough_wavefronts_stream(lib, shape, step, phase, slices):
    """With fewer K-slices a wavefront takes a whole tile: where there are few tiles, eight slices stream wider."""
    dtype, hidden, ffn, heads, kv = shape
    batch, n_new, k = step
    cfg = B.make_config(small_shape(dtype, hidden=hidden, n_heads=heads, n_kv_heads=kv, head_dim=128, ffn=ffn, vocab=2069), max_batch=batch,
                        max_new=n_new, max_positions=512, max_topk=8, k_max=k)
    st, plans = _plan(lib, cfg, batch, n_new, k)
    assert st == B.PS_OK
    _check_plan(cfg, plans, batch, n_new, k, 256, 160 * 1024)
    p = plans[phase]
    streaming = p["T"] * (1 << p["s_log"] + p["kw_log"]) / (p["rounds"] * 256 * PS_WAVES)
    assert 1 << p["s_log"] == slices and streaming >= 0.25, (p, streaming)


def _weight_bytes(cfg):
    qd, esz = cfg.n_heads * cfg.head_dim, 2 if cfg.dtype == B.PS_BF16 else 4
    kv = cfg.n_kv_heads * cfg.head_dim
    return esz * cfg.hidden * (qd + 2 * kv + qd + 3 * cfg.ffn + 16 * -(-cfg.vocab // 16))


def test_step_plans_choose_the_workgroups_of_small_steps(lib):
    """The whole plan of a step as ps_draft_step makes it: five workgroups for every eight compute units below 48 KB of
    weights per compute unit, up to 32 rows and as long as the attention does not need the others; on both sides of each limit."""
    def nwg(shape, kv, n_new, k, n_cu=256, lds=160 * 1024):
        cfg = B.make_config(shape, max_batch=len(kv), max_new=n_new, max_positions=1 << 16, max_topk=8, k_max=max(k, 1))
        st, n, plans, attn = DBG.ps_draft_debug_step_plan(cfg, kv, n_new, k, 0, n_cu, lds)
        assert st == B.PS_OK
        _check_plan(cfg, plans, len(kv), n_new, k, n, lds)
        return n
    bf, tiny = small_shape("bf16"), WORKLOADS["c0"].shape
    assert nwg(bf, [100], 1, 4) == 160 and nwg(bf, [100], 1, 4, n_cu=304) == 190 and nwg(bf, [100], 1, 4, n_cu=7) == 7
    assert nwg(bf, [100] * 8, 1, 3) == 160 and nwg(bf, [100] * 11, 1, 2) == 256                   # 32 and 33 rows
    for vocab, n in ((5136, 160), (6160, 256)):                                                   # 44 and 48.2 KB of weights per compute unit
        assert nwg(small_shape("bf16", vocab=vocab), [100], 1, 4) == n, vocab
    assert nwg(small_shape("f32"), [100], 1, 4) == 256
    for kv, n_new, k, n in (([4000], 1, 4, 160), ([8000], 1, 4, 256),                             # float32: one round of blocks of 128 keys, ...
                            ([1024] * 4, 1, 4, 160), ([2048] * 4, 1, 4, 256),                     # ... or the step's rows left to the merge items for it
                            ([512] * 6, 1, 4, 160), ([1024] * 6, 1, 4, 256), ([2048] * 6, 1, 4, 256),
                            ([256] * 16, 1, 1, 160), ([600] * 16, 1, 1, 256), ([300] * 32, 1, 0, 256)):
        assert nwg(tiny, kv, n_new, k) == n, (kv, n_new, k)
    for kv, n_new, k, n in (([4096], 1, 4, 160), ([1024] * 4, 1, 4, 160), ([2048] * 6, 1, 4, 160),     # bf16: the same or up to a third more
                            ([4096] * 6, 1, 4, 256), ([1024] * 32, 1, 0, 256), ([2048] * 32, 1, 0, 256)):   # half as much more; another round
        assert nwg(bf, kv, n_new, k) == n, (kv, n_new, k)
    cfg = B.make_config(tiny, max_batch=1, max_new=1, max_positions=128, max_topk=4, k_max=4)
    for kw, want in ((dict(n_cu=0), B.PS_ERR_SHAPE), (dict(n_cu=513), B.PS_ERR_SHAPE), (dict(kv=(124,)), B.PS_ERR_KV_CAPACITY), (dict(k=5), B.PS_ERR_SHAPE)):
        a = dict(dict(kv=(64,), k=4, n_cu=256), **kw)
        assert DBG.ps_draft_debug_step_plan(cfg, a["kv"], 1, a["k"], 0, a["n_cu"], 160 * 1024)[0] == want, kw


def test_step_plans_over_a_sweep_of_small_shapes(lib):
    """Random small shapes, batches, lengths and devices: the phase plans hold for the number of workgroups that was chosen
    (what the device code relies on), that number is one of the two, and the attention's work covers every sequence."""
    import random
    rnd = random.Random(19)
    chosen = {"all": 0, "fewer": 0}
    for _ in range(600):
        dtype = rnd.choice(["bf16", "f32"])
        head_dim, n_kv, grp = rnd.choice([64, 128]), rnd.choice([1, 2, 4]), rnd.choice([1, 2, 4])
        mul = 32 if dtype == "bf16" else 16
        shape = small_shape(dtype, hidden=n_kv * grp * head_dim, n_heads=n_kv * grp, n_kv_heads=n_kv, head_dim=head_dim,
                            ffn=mul * rnd.randint(1, 60), vocab=rnd.randint(16, 9000))
        k, n_new = rnd.randint(0, 8), rnd.randint(1, 6)
        M = n_new + k
        if grp * M > 64:
            continue
        batch = rnd.randint(1, max(1, min(32, 64 // M)))
        kv = [rnd.choice([0, 1, 127, 128, 129, rnd.randint(0, 3000)]) for _ in range(batch)]
        cfg = B.make_config(shape, max_batch=batch, max_new=n_new, max_positions=4096, max_topk=8, k_max=max(k, 1))
        for n_cu, lds in ((256, 160 * 1024), (304, 160 * 1024), (80, 64 * 1024), (8, 96 * 1024), (7, 96 * 1024)):
            st, n, plans, attn = DBG.ps_draft_debug_step_plan(cfg, kv, n_new, k, rnd.randint(0, 1), n_cu, lds)
            assert st in (B.PS_OK, B.PS_ERR_UNSUPPORTED), (st, kv)
            if st != B.PS_OK:
                continue
            tag = (dtype, kv, n_new, k, n_cu, n, attn)
            assert n in (n_cu, n_cu * 5 // 8 if n_cu >= 8 else n_cu), tag
            small = batch * M <= 32 and _weight_bytes(cfg) <= n_cu * 48 * 1024     # (the packed bytes are these, rounded up)
            assert n == n_cu or small, tag
            chosen["all" if n == n_cu else "fewer"] += 1
            _check_plan(cfg, plans, batch, n_new, k, n, lds)
            blocks = n_kv * sum(max(1, -(-l // attn["keys"])) if dtype == "bf16" else -(-(l + (0 if attn["sep"] else M)) // attn["keys"]) for l in kv)
            passes = -(-grp * M // 16) if dtype == "bf16" else 1
            assert attn["blocks"] == blocks and attn["units"] == blocks * passes, tag
            assert attn["workgroups"] == min(n, max(attn["units"], attn["merge_items"])), tag
            if dtype == "f32" and n < n_cu:
                assert attn["units"] <= n or -(-attn["units"] // n) <= -(-attn["units"] // n_cu), tag
    assert min(chosen.values()) > 100, chosen


def _keys_left(g, lists, topk, per_list, log):
    """Keys that the lower bound of lm_merge_row leaves, on a row of normally distributed logits: the topk-th largest of the
    groups' largest (all keys of the lists if there are fewer groups)."""
    x = np.sort(g.standard_normal((lists, per_list)), axis=1)[:, ::-1][:, :topk]
    top = np.sort([x[i:i + (1 << log), 0].max() for i in range(0, lists, 1 << log)])[::-1]
    return int((x >= top[topk - 1]).sum()) if len(top) >= topk else x.size


def test_the_row_merge_selects_only_where_the_bound_leaves_few_keys(lib):
    """A row whose bound leaves more than 64 keys pays for the selection and the merge: at most 1.2 % of rows of normally distributed
    logits by the counts that the rule was made from, so (five standard deviations) at most 14 of 400, on both sides of every
    limit of the number of lists; at most 64 groups; and rows are selected wherever there are more lists than keys."""
    g = np.random.default_rng(17)
    for topk in range(1, 33):
        for lists in (1, 4, 5, 7, 8, 10, 11, 12, 13, 14, 16, 17, 18, 20, 31, 32, 33, 38, 39, 40, 50, 64, 65, 68, 72, 80, 128, 129, 137, 150, 160, 256, 257, 304, 512):
            log = DBG.ps_draft_debug_merge_groups(lists, topk)
            if not 5 <= topk <= 16:
                assert log == -1, (lists, topk, log)
            if log < 0:
                assert topk < 5 or topk > 16 or lists <= topk, (lists, topk, log)
                continue
            assert -(-lists // (1 << log)) <= 64, (lists, log)
            many = sum(_keys_left(g, lists, topk, 16, log) > 64 for _ in range(400 if topk >= 12 else 20))
            assert many <= 14, (lists, topk, log, many)
