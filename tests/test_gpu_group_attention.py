"""GPU parity of the group-wise training attention (Section 4.1) through the C ABI against the CPU oracle,
element by element.  Tolerance: the kernel accumulates in float32 with queries split into bf16 high and low
parts (about 1e-5 relative); keys are rounded to the storage type after the rotary embedding on both sides, so
where the float32 and the float64 rotation fall on different sides of a rounding boundary a key moves by one
unit in the last place (bf16: 2^-8 of one element of one key), which moves a score by up to ~1e-2 |q_j k_j| /
sqrt(d) and an output by a few 1e-4: outputs are compared to 2e-3 (bf16) / 2e-5 (f32) of the largest value."""
import numpy as np
import pytest

from oracle import group_attention as ga
from paper_2410_05589_amd import binding as B
from paper_2410_05589_amd import debug as DBG
from paper_2410_05589_amd import inputs
from paper_2410_05589_amd import train as TR

pytestmark = pytest.mark.gpu

# The kernels as ps_train_debug_launch numbers them: float32 with 64 rows x 2 wavefronts per 16 (head_dim 128), bf16 tiles of 16
# rows, bf16 blocks of 128 rows, float32 with 32 rows x 2 (head_dim 64), float32 with 32 rows x 4 (short calls)
F32_64, TILES, WIDE, F32_32, F32_SHORT = range(5)


def check_kernel(want, seqs, T, k, nq, nkv, d, dtype):
    st, g = DBG.ps_train_debug_launch(TR.make_args(seqs, T, k, nq, nkv, d, dtype, 10000.0))
    assert st == B.PS_OK and g["kernel"] == want, g


def run_gpu(inp, seqs, T, k, nq, nkv, d, dtype, base=10000.0):
    import torch
    a = TR.make_args(seqs, T, k, nq, nkv, d, dtype, base)
    q, kk, v = (B.to_device(inp[n], dtype) for n in ("q", "k", "v"))
    out = torch.full((seqs, T * (k + 1), nq, d), -12345.0, dtype=torch.float32, device="cuda:0")
    ws = torch.empty(TR.ps_group_attention_workspace_bytes(a) + 256, dtype=torch.uint8, device="cuda:0")
    a.q, a.k_, a.v, a.out = q.data_ptr(), kk.data_ptr(), v.data_ptr(), out.data_ptr()
    a.workspace = (ws.data_ptr() + 255) & ~255
    a.workspace_bytes = ws.numel() - 256
    st = TR.ps_group_attention(a, torch.cuda.current_stream().cuda_stream)
    assert st == B.PS_OK, B.ps_draft_strerror(st)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _case(seqs, T, k, nq, nkv, d, dtype, seed, base=10000.0, kernel=None):
    if kernel is not None:
        check_kernel(kernel, seqs, T, k, nq, nkv, d, dtype)
    print("case seqs", seqs, "T", T, "k", k, "heads", nq, nkv, "d", d, dtype, flush=True)
    inp = inputs.make_group_attention_inputs(seed, seqs, T, k, nq, nkv, d, dtype)
    got = run_gpu(inp, seqs, T, k, nq, nkv, d, dtype, base)
    worst = 0.0
    for s in range(seqs):
        want = ga.group_attention(inp["q"][s], inp["k"][s], inp["v"][s], T, k, base, dtype)
        err = float(np.abs(got[s] - want).max())
        worst = max(worst, err)
        assert err <= (2e-5 if dtype == "f32" else 2e-3) * np.abs(want).max(), (s, err)
    print("    max abs error", worst, flush=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_small_shapes_ragged_tiles(dtype):
    _case(2, 37, 4, 4, 2, 64, dtype, 1)          # blocks that end inside a group, a ragged last block, GQA
    _case(1, 50, 2, 2, 2, 128, dtype, 2)
    _case(1, 21, 7, 2, 1, 64, dtype, 3)          # groups that divide the blocks' rows
    _case(1, 9, 15, 2, 2, 64, dtype, 4)          # the longest groups
    _case(1, 70, 0, 4, 4, 64, dtype, 5)          # k = 0: ordinary causal attention
    _case(1, 1, 4, 2, 2, 64, dtype, 6)           # a single token


def test_longer_sequence_and_other_rope_base_bf16():
    _case(1, 300, 4, 8, 2, 128, "bf16", 7, base=500000.0)


@pytest.mark.parametrize("base", [2.0, 1.0, 2.0 ** -24])
def test_rotary_bases_that_reach_large_angles(base):
    """base 2: every pair turns many times; 1: all alike; 2^-24: angles up to 1.6e9, beyond the range that the table's own cosine and
    sine reduce.  The call takes the base as float32, so these are numbers that it holds exactly (1e-7 is not: half a unit in its last
    place turns an angle of 1e9 by 30); an angle of 1.6e9 is then known to 1.6e9 * 2^-52 = 4e-7 on either side."""
    _case(1, 150, 3, 2, 1, 64, "f32", 12, base=base)


@pytest.mark.parametrize("base", [2.0, 1.0, 2.0 ** -24])
@pytest.mark.parametrize("T,k,d", [(150, 0, 128), (150, 0, 64), (97, 1, 64), (60, 8, 128)])
def test_rotary_bases_that_reach_large_angles_in_the_wide_kernel(T, k, d, base):
    """The same where the wide kernel takes a wavefront's (k = 0) or a workgroup's part of the table through LDS."""
    _case(1, T, k, 2, 1, d, "bf16", 13, base=base, kernel=WIDE)


@pytest.mark.parametrize("T,d,base", [(1 << 17, 64, 2.0), (1 << 17, 128, 10.0), (1 << 17, 128, 10000.0), (1 << 17, 64, 500000.0), (1 << 20, 64, 1000000.0)])
def test_entries_of_the_rotary_table(T, d, base):
    """The table (first in the workspace) against cosines and sines in extended precision: half a unit in the last place of the float
    that is nearest, and what two units in the last place of the angle in double precision turn; and nearly all entries are that float."""
    import torch
    a = TR.make_args(1, T, 0, 1, 1, d, "bf16", base)
    x = torch.zeros((T, 1, d), dtype=torch.bfloat16, device="cuda:0")
    out = torch.empty((T, 1, d), dtype=torch.float32, device="cuda:0")
    nbytes = TR.ps_group_attention_workspace_bytes(a)
    ws = torch.full((nbytes + 256,), 0xFF, dtype=torch.uint8, device="cuda:0")
    a.q = a.k_ = a.v = x.data_ptr()
    a.out = out.data_ptr()
    a.workspace, a.workspace_bytes = (ws.data_ptr() + 255) & ~255, nbytes
    print("case table T", T, "d", d, "base", base, flush=True)
    assert TR.ps_group_attention(a, torch.cuda.current_stream().cuda_stream) == B.PS_OK
    torch.cuda.synchronize()
    lo = a.workspace - ws.data_ptr()
    tab = ws[lo:lo + T * d * 4].cpu().numpy().view(np.float32).reshape(T, d // 2, 2)
    g = np.random.default_rng(5)
    pos = np.unique(np.concatenate([np.arange(300), g.integers(0, T, 3000), np.arange(T - 100, T)]))
    ld = np.longdouble
    ang = pos.astype(ld)[:, None] * np.exp2(-ld(2) * np.arange(d // 2).astype(ld) / ld(d) * np.log2(ld(base)))[None, :]
    want = np.stack([np.cos(ang), np.sin(ang)], axis=2)
    near = want.astype(np.float32)
    err = np.abs(tab[pos].astype(ld) - want)
    assert (err <= np.spacing(np.abs(near)) / 2 + ang[:, :, None] * ld(2.0 ** -51) + ld(2.0 ** -53)).all(), float(err.max())
    other = int((tab[pos] != near).sum())
    print("    not the nearest float:", other, "of", near.size, "largest error", float(err.max()), flush=True)
    assert other <= near.size // 1000


@pytest.mark.parametrize("T,k,d", [(40, 14, 128), (45, 12, 64), (50, 8, 128), (50, 10, 64)])
def test_own_keys_in_both_tiles_whose_scores_lie_far_apart(T, k, d):
    """The wide kernel gives the own [MASK] keys of a wavefront's rows and of the 16 rows before one reference.  Keys 32 times as long: the
    scores of a row spread over a hundred and more, and where the largest leads by 20 the output is its value row (what is left weighs
    below T e^-20; a key that rounds the other way moves a score by less than 1), in whichever tile it stands."""
    from oracle.ps_oracle import round_to_storage, widen
    check_kernel(WIDE, 1, T, k, 8, 8, d, "bf16")
    inp = inputs.make_group_attention_inputs(17, 1, T, k, 8, 8, d, "bf16")
    inp["k"] = round_to_storage(32.0 * widen(inp["k"], "bf16"), "bf16")
    print("case far apart T", T, "k", k, "d", d, flush=True)
    got = run_gpu(inp, 1, T, k, 8, 8, d, "bf16")[0]
    _, probs = ga.group_attention(inp["q"][0], inp["k"][0], inp["v"][0], T, k, 10000.0, "bf16", return_probs=True)
    v = widen(inp["v"][0], "bf16")
    order = np.sort(probs, axis=2)
    won = probs.argmax(axis=2)
    i, h = np.nonzero(order[:, :, -2] < np.exp(-20.0))
    w = won[i, h]
    own = (w % (k + 1) > 0)
    before = own & (w // 32 < i // 32)
    print("    rows:", len(i), "own key:", int(own.sum()), "in the tile before:", int(before.sum()), flush=True)
    assert own.sum() >= 100 and before.sum() >= 10
    assert np.abs(got[i, h] - v[w, h]).max() <= 1e-5 * np.abs(v).max()


def test_longer_sequences_with_other_group_sizes():
    """Several tiles of keys per wavefront (tiles every query sees entirely, the masked last ones, the own [MASK] rows), several
    blocks of rows, with 8, 16 and 2 rows per group in the wide bf16 kernel and 4 in the float32 one of short calls."""
    _case(1, 200, 7, 4, 4, 128, "bf16", 8)
    _case(1, 130, 15, 2, 1, 128, "bf16", 9)
    _case(2, 150, 1, 4, 2, 64, "bf16", 10)
    _case(1, 120, 3, 4, 4, 128, "f32", 11)


@pytest.mark.parametrize("seqs,T,k,nq,nkv,d", [
    (1, 33, 0, 2, 2, 128), (1, 128, 0, 2, 1, 64), (1, 129, 0, 1, 1, 128),     # k = 0 (no own rows): 1, exactly 1 and 2 blocks of 128 rows
    (1, 64, 1, 2, 2, 128), (2, 65, 1, 3, 1, 64),                              # two rows per group: the most positions in a block; 1 and 2 blocks
    (1, 43, 2, 2, 2, 64), (1, 96, 2, 3, 3, 128),                              # blocks that start inside a group; rows = 129, 288
    (1, 33, 4, 2, 1, 128), (2, 51, 4, 2, 2, 64), (1, 33, 8, 4, 2, 128),       # just above 32 tokens
    (1, 33, 15, 2, 2, 128), (1, 40, 10, 3, 3, 64), (3, 16, 3, 5, 1, 128),     # 16 rows per group; a wavefront without rows; 15 heads x sequences
    (1, 32, 4, 2, 2, 128), (1, 32, 15, 2, 1, 64)])                            # 32 tokens, on either side of the 16-row kernel's range
def test_blocks_of_128_rows_at_their_edges(seqs, T, k, nq, nkv, d):
    _case(seqs, T, k, nq, nkv, d, "bf16", 100 + T + k)


@pytest.mark.parametrize("seqs,T,k,nq,nkv,d", [
    (1, 1, 4, 2, 1, 128), (2, 1, 15, 2, 2, 64), (1, 31, 4, 4, 2, 128), (2, 32, 5, 2, 1, 64),   # 3 and 2 groups per tile, a ragged last tile
    (1, 32, 14, 2, 2, 128), (3, 17, 10, 4, 4, 64),                                             # one group per tile
    (1, 32, 8, 32, 8, 64), (1, 32, 7, 2, 2, 128), (1, 26, 8, 36, 36, 64)])                     # 256 workgroups; two calls of the wide kernel
def test_tiles_of_16_rows_at_their_edges(seqs, T, k, nq, nkv, d):
    _case(seqs, T, k, nq, nkv, d, "bf16", 300 + T + k)


@pytest.mark.parametrize("seqs,T,k,nq,nkv,d", [
    (1, 64, 0, 2, 1, 64), (1, 65, 0, 1, 1, 128),                  # k = 0: exactly 2 blocks of 32 rows and one more row; 1 and 2 stages of 64 keys
    (1, 33, 1, 2, 2, 64), (2, 43, 2, 3, 1, 64),                   # blocks that start inside a group; a query tile without rows
    (1, 13, 4, 2, 2, 128), (1, 40, 10, 2, 1, 64), (3, 17, 15, 2, 2, 64),
    (1, 32, 0, 1, 1, 64), (1, 33, 0, 2, 1, 64), (1, 64, 0, 1, 1, 128), (2, 65, 0, 1, 1, 64),   # exactly 1, 2 and 3 blocks of 32 rows
    (1, 9, 7, 2, 2, 64), (1, 5, 15, 2, 1, 128), (1, 1, 2, 1, 1, 64),                            # own rows of several stages; a wavefront without keys
    (1, 88, 7, 32, 8, 64), (1, 100, 7, 16, 16, 128)])                                           # the longest short calls: 704 and 400 blocks
def test_float32_short_calls_at_their_edges(seqs, T, k, nq, nkv, d):
    _case(seqs, T, k, nq, nkv, d, "f32", 200 + T + k, kernel=F32_SHORT)


@pytest.mark.parametrize("seqs,T,k,nq,nkv,d", [
    (8, 64, 0, 46, 23, 64), (8, 65, 0, 30, 30, 64),               # k = 0: exactly 2 blocks of 32 rows, and one more row; 2 and 3 stages of 32 keys
    (12, 33, 1, 20, 4, 64), (10, 43, 2, 15, 5, 64),               # blocks that start inside a group; a query tile without rows
    (8, 13, 4, 32, 8, 64), (6, 40, 10, 9, 3, 64), (8, 17, 15, 10, 10, 64), (24, 1, 2, 30, 1, 64), (5, 5, 15, 50, 25, 64),
    (5, 150, 3, 8, 8, 64),
    (7, 64, 0, 30, 15, 128), (7, 65, 0, 20, 20, 128), (7, 129, 0, 12, 3, 128),   # blocks of 64 rows: exactly 1, one more row, exactly 2 and one more
    (7, 33, 1, 20, 4, 128), (6, 43, 2, 15, 5, 128), (5, 13, 4, 28, 7, 128), (4, 40, 10, 9, 3, 128), (5, 17, 15, 10, 10, 128),
    (16, 1, 2, 26, 1, 128), (4, 5, 15, 40, 20, 128), (4, 100, 3, 8, 4, 128)])
def test_float32_longer_calls_at_their_edges(seqs, T, k, nq, nkv, d):
    """Calls beyond the short ones (704 workgroups of 32 rows, head_dim 128: 400): 32 rows with two wavefronts per 16, 64 rows for head_dim 128."""
    _case(seqs, T, k, nq, nkv, d, "f32", 300 + T + k, kernel=F32_32 if d == 64 else F32_64)


@pytest.mark.parametrize("dtype,k,nq,d,kernel", [
    ("bf16", 0, 2, 128, WIDE), ("bf16", 0, 2, 64, WIDE), ("bf16", 3, 2, 128, WIDE), ("f32", 0, 2, 64, F32_SHORT), ("f32", 3, 2, 128, F32_SHORT),
    ("f32", 0, 240, 64, F32_32), ("f32", 3, 80, 64, F32_32), ("f32", 0, 140, 128, F32_64), ("f32", 3, 46, 128, F32_64)])
def test_scores_that_overflow_before_a_row_sees_a_finite_one(dtype, k, nq, d, kernel):
    """The first 32 real tokens' keys lie opposite to every query and so far out that their scores are -inf in float32
    (q.k = -1e40; in the pair of dimensions that the rotation turns least); from token 32 on all keys are ordinary.  Rows
    that see an ordinary real token have a finite result, the oracle's (float64: the first 32 weigh exp(-1e39) = 0)."""
    T = 70
    print("case overflowing scores", dtype, "k", k, "heads", nq, "d", d, flush=True)
    check_kernel(kernel, 1, T, k, nq, nq, d, dtype)
    inp = inputs.make_group_attention_inputs(31 + k, 1, T, k, nq, nq, d, dtype)
    from oracle.ps_oracle import round_to_storage, widen
    q, kk = widen(inp["q"], dtype), widen(inp["k"], dtype)
    j = d // 2 - 1
    q[...] = 0.0
    q[..., j] = 1e20
    kk[:, :32 * (k + 1)] = 0.0
    kk[:, :32 * (k + 1), :, j] = -1e20
    kk[:, 32 * (k + 1):, :, j] *= 1e-20
    kk[:, 32 * (k + 1):, :, d - 1] *= 1e-20
    inp["q"], inp["k"] = round_to_storage(q, dtype), round_to_storage(kk, dtype)
    got = run_gpu(inp, 1, T, k, nq, nq, d, dtype)[0]
    want = ga.group_attention(inp["q"][0], inp["k"][0], inp["v"][0], T, k, 10000.0, dtype)
    rows = slice(32 * (k + 1), None)
    assert np.isfinite(got[rows]).all()
    assert np.abs(got[rows] - want[rows]).max() <= (2e-3 if dtype == "bf16" else 2e-5) * np.abs(want[rows]).max()


@pytest.mark.parametrize("dtype,T,k,nq,nkv,d,kernel", [
    ("bf16", 70, 4, 2, 1, 128, WIDE), ("bf16", 70, 4, 2, 2, 64, WIDE), ("bf16", 150, 0, 2, 2, 128, WIDE), ("bf16", 40, 15, 2, 2, 64, WIDE),
    ("f32", 70, 4, 2, 1, 64, F32_SHORT), ("f32", 90, 0, 2, 2, 128, F32_SHORT), ("f32", 20, 15, 2, 2, 64, F32_SHORT),
    ("f32", 70, 4, 66, 11, 64, F32_32), ("f32", 90, 0, 236, 59, 64, F32_32), ("f32", 20, 15, 72, 72, 64, F32_32),
    ("f32", 70, 4, 38, 19, 128, F32_64), ("f32", 90, 0, 134, 67, 128, F32_64), ("f32", 20, 15, 42, 42, 128, F32_64),
    ("bf16", 20, 5, 2, 2, 128, TILES), ("bf16", 32, 14, 2, 2, 64, TILES),
    ("bf16", 32, 15, 2, 2, 64, WIDE)])
def test_values_that_a_row_may_not_see_do_not_reach_it(dtype, T, k, nq, nkv, d, kernel):
    """Value rows that hold Inf and NaN: two [MASK] tokens' and one real token's.  Rows that see none of them have the
    oracle's result (their own keys and values only), the others are not finite."""
    from oracle.ps_oracle import widen
    print("case non-finite values", dtype, "T", T, "k", k, "heads", nq, nkv, "d", d, flush=True)
    check_kernel(kernel, 1, T, k, nq, nkv, d, dtype)
    inp = inputs.make_group_attention_inputs(61 + T + k, 1, T, k, nq, nkv, d, dtype)
    want = ga.group_attention(inp["q"][0], inp["k"][0], inp["v"][0], T, k, 10000.0, dtype)
    K1 = k + 1
    poison = [((T // 4) * K1 + k // 2, np.inf), ((T // 2 + 1) * K1 + k, np.nan), ((2 * T // 3) * K1, -np.inf)]
    v = widen(inp["v"], dtype)
    for row, x in poison:
        v[0, row] = x
    if dtype == "bf16":
        bits = v.astype(np.float32).view(np.uint32) >> np.uint32(16)
        inp["v"] = bits.astype(np.uint16)
    else:
        inp["v"] = v.astype(np.float32)
    got = run_gpu(inp, 1, T, k, nq, nkv, d, dtype)[0]
    vis = ga.group_mask(T, k)
    sees = vis[:, [row for row, _ in poison]].any(axis=1)
    assert sees.any() and not sees.all()
    assert not np.isfinite(got[sees]).any()
    assert np.abs(got[~sees] - want[~sees]).max() <= (2e-3 if dtype == "bf16" else 2e-5) * np.abs(want).max()


@pytest.mark.parametrize("dtype,T,k,nq,nkv,d,kernel", [
    ("bf16", 90, 4, 4, 2, 128, WIDE), ("bf16", 70, 0, 2, 2, 64, WIDE), ("bf16", 20, 5, 2, 2, 128, TILES), ("f32", 50, 3, 4, 2, 64, F32_SHORT),
    ("f32", 40, 2, 6, 3, 128, F32_SHORT), ("f32", 50, 3, 104, 52, 64, F32_32), ("f32", 50, 3, 60, 30, 128, F32_64)])
def test_tensors_that_are_aligned_to_four_bytes_only(dtype, T, k, nq, nkv, d, kernel):
    """q, k, v and out at 4, 8 and 12 bytes from a 16-byte boundary: the outputs of the same call with aligned ones."""
    import torch
    print("case alignment", dtype, "T", T, "k", k, "heads", nq, nkv, "d", d, flush=True)
    check_kernel(kernel, 1, T, k, nq, nkv, d, dtype)
    inp = inputs.make_group_attention_inputs(91, 1, T, k, nq, nkv, d, dtype)
    want = run_gpu(inp, 1, T, k, nq, nkv, d, dtype)
    esz = 2 if dtype == "bf16" else 4
    for shift in (4, 8, 12):
        a = TR.make_args(1, T, k, nq, nkv, d, dtype, 10000.0)
        t = {}
        for n in ("q", "k", "v"):
            x = B.to_device(inp[n], dtype).reshape(-1)
            t[n] = torch.empty(x.numel() + 16 // esz, dtype=x.dtype, device="cuda:0")[shift // esz:shift // esz + x.numel()]
            t[n].copy_(x)
        out = torch.full((want.size + 4,), -12345.0, dtype=torch.float32, device="cuda:0")
        o = out[shift // 4:shift // 4 + want.size]
        assert all(x.data_ptr() % 16 == shift for x in (t["q"], t["k"], t["v"], o))
        ws = torch.empty(TR.ps_group_attention_workspace_bytes(a) + 256, dtype=torch.uint8, device="cuda:0")
        a.q, a.k_, a.v, a.out = t["q"].data_ptr(), t["k"].data_ptr(), t["v"].data_ptr(), o.data_ptr()
        a.workspace, a.workspace_bytes = (ws.data_ptr() + 255) & ~255, ws.numel() - 256
        assert TR.ps_group_attention(a, torch.cuda.current_stream().cuda_stream) == B.PS_OK
        torch.cuda.synchronize()
        assert np.array_equal(o.cpu().numpy().reshape(want.shape), want), shift
        rest = torch.cat([out[:shift // 4], out[shift // 4 + want.size:]])
        assert bool((rest == -12345.0).all()), shift


def test_more_workgroups_than_one_dimension_of_a_launch_holds():
    """4097 one-token sequences of 4096 heads: 2^24 + 4096 workgroups of 256 work items.  Each row sees itself only, so
    every head's output is the sequence's value row, exactly."""
    import torch
    seqs, nq, d = 4097, 4096, 64
    print("case seqs", seqs, "heads", nq, flush=True)
    a = TR.make_args(seqs, 1, 0, nq, 1, d, "bf16", 10000.0)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    q = torch.randn((seqs, 1, nq, d), generator=g, device="cuda:0", dtype=torch.bfloat16)
    kk, v = (torch.randn((seqs, 1, 1, d), generator=g, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
    out = torch.full((seqs, 1, nq, d), -12345.0, dtype=torch.float32, device="cuda:0")
    ws = torch.empty(TR.ps_group_attention_workspace_bytes(a) + 256, dtype=torch.uint8, device="cuda:0")
    a.q, a.k_, a.v, a.out = q.data_ptr(), kk.data_ptr(), v.data_ptr(), out.data_ptr()
    a.workspace, a.workspace_bytes = (ws.data_ptr() + 255) & ~255, ws.numel() - 256
    st = TR.ps_group_attention(a, torch.cuda.current_stream().cuda_stream)
    assert st == B.PS_OK, B.ps_draft_strerror(st)
    torch.cuda.synchronize()
    assert bool((out == v.float()).all())


def test_the_error_is_the_rounding_of_the_rotated_keys():
    """The tolerance above is spent on keys that round the other way after a float32 rotation (the kernel's) than
    after a float64 rotation (the oracle's).  With the keys rotated in float32 on the CPU, as the kernel's key
    rotation does it, and everything else as in the oracle (float64), the outputs agree to float32 accuracy."""
    from oracle.ps_oracle import rope, round_to_storage, widen
    seqs, T, k, nq, nkv, d, dtype, seed = 1, 49, 7, 12, 3, 64, "bf16", 1039
    inp = inputs.make_group_attention_inputs(seed, seqs, T, k, nq, nkv, d, dtype)
    got = run_gpu(inp, seqs, T, k, nq, nkv, d, dtype)[0]
    want = ga.group_attention(inp["q"][0], inp["k"][0], inp["v"][0], T, k, 10000.0, dtype)
    Q, K, V = widen(inp["q"][0], dtype), widen(inp["k"][0], dtype), widen(inp["v"][0], dtype)
    _, _, pos = ga.group_layout(T, k)
    half = d // 2
    ang = pos[:, None].astype(np.float64) * np.exp(-2.0 * np.arange(half) / d * np.log(10000.0))[None, :]
    cs, sn = np.cos(ang).astype(np.float32)[:, None, :], np.sin(ang).astype(np.float32)[:, None, :]
    a, b = K.astype(np.float32)[:, :, :half], K.astype(np.float32)[:, :, half:]
    k32 = np.concatenate([a * cs - b * sn, b * cs + a * sn], axis=2)            # float32 arithmetic, pairs (j, j + d/2)
    Kr = widen(round_to_storage(k32.astype(np.float64), dtype), dtype)
    K64 = widen(round_to_storage(rope(K, pos, 10000.0), dtype), dtype)
    print("    keys that round differently:", int((Kr != K64).sum()), "of", Kr.size, flush=True)
    Qr, vis, grp = rope(Q, pos, 10000.0), ga.group_mask(T, k), nq // nkv
    exp32 = np.zeros_like(want)
    for i in range(want.shape[0]):
        cols = np.nonzero(vis[i])[0]
        for h in range(nq):
            s = Kr[cols, h // grp, :] @ Qr[i, h, :] / np.sqrt(d)
            p = np.exp(s - s.max())
            exp32[i, h, :] = (p / p.sum()) @ V[cols, h // grp, :]
    e_oracle, e_32 = np.abs(got - want).max(), np.abs(got - exp32).max()
    print("    error against the oracle", e_oracle, "against the float32-rotated keys", e_32, flush=True)
    assert e_oracle <= 2e-3 * np.abs(want).max()
    assert e_32 <= 2e-5 * np.abs(want).max()


def test_sampled_rows_at_the_benchmark_size():
    """T 2048, k 4, 32 heads x 128 (the 7B drafter's layer), bf16: rows the oracle works out one by one."""
    T, k, nq, d = 2048, 4, 32, 128
    inp = inputs.make_group_attention_inputs(8, 1, T, k, nq, nq, d, "bf16")
    got = run_gpu(inp, 1, T, k, nq, nq, d, "bf16")
    from oracle.ps_oracle import rope, round_to_storage, widen
    g = np.random.default_rng(0)
    rows = sorted(set([0, 1, 4, 5, T * (k + 1) - 1, T * (k + 1) - 5] + [int(x) for x in g.integers(0, T * (k + 1), 10)]))
    heads = [0, 13, 31]
    pos_all = np.arange(T * (k + 1)) // (k + 1) + np.arange(T * (k + 1)) % (k + 1)
    K = {h: widen(round_to_storage(rope(widen(inp["k"][0][:, h:h + 1], "bf16"), pos_all, 10000.0), "bf16"), "bf16")[:, 0] for h in heads}
    for i in rows:
        gi, si = divmod(i, k + 1)
        cols = [gg * (k + 1) for gg in range(gi + 1)] + [gi * (k + 1) + ss for ss in range(1, si + 1)]   # what the row may see
        for h in heads:
            qv = rope(widen(inp["q"][0][i:i + 1, h:h + 1], "bf16"), pos_all[i:i + 1], 10000.0)[0, 0]
            s = K[h][cols] @ qv / np.sqrt(d)
            p = np.exp(s - s.max())
            want = (p / p.sum()) @ widen(inp["v"][0][cols, h], "bf16")
            err = float(np.abs(got[0, i, h] - want).max())
            assert err <= 2e-3 * max(1.0, np.abs(want).max()), (i, h, err)
    # property at any size: every output row is a convex combination of value rows
    assert np.isfinite(got).all() and np.abs(got).max() <= np.abs(widen(inp["v"], "bf16")).max() + 1e-3
