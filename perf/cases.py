"""What the performance of this framework is measured on: the work a speculative decoder with a parallel drafter, and
the training of that drafter, has the library do through its public entry points.

Three kinds of cases:
  draft   ps_draft_step: one parallel draft step (a decode step of 1 .. n_new accepted tokens plus k [MASK] slots
          against the KV cache, LM head with softmax and top-k): every drafter shape of paper_2410_05589_amd/configs.py
          and the small one of the tests, one sequence and batches, hidden states / token ids / token ids + target
          features as input, sequences that accepted different numbers of tokens, sampling and full probabilities
  verify  ps_tree_tokens + ps_verify_walk: what follows the step in a round, the draft tree's tokens (the target model
          needs them) and the acceptance walk against the target's distributions
  train   ps_group_attention: the attention of a training sequence laid out as parallel groups

A state holds the weights and the context of one drafter as a serving program keeps them, the argument structures, the
inputs and the output buffers; one pass is the call (a walk: the two calls), asynchronous, on the current stream.
Values follow paper_2410_05589_amd/inputs.py: matrices and cached K/V ~ N(0, 0.02), gains 1 + N(0, 0.02), hidden
states, embeddings and training q, k, v ~ N(0, 1); peaked distributions for the walk.
"""
import ctypes
import math

import torch

from paper_2410_05589_amd import binding as B
from paper_2410_05589_amd import train as TR
from paper_2410_05589_amd import verify as VF
from paper_2410_05589_amd.configs import WORKLOADS, small_shape
from paper_2410_05589_amd.inputs import draft_tree

DEVICE = "cuda:0"

SHAPES = {
    "tiny": WORKLOADS["c0"].shape,             # float32, H 256, 4 heads x 64
    "small": small_shape("bf16"),              # H 512, 8 heads x 64, V 2064
    "small_f32": small_shape("f32"),
    "7b": WORKLOADS["c1"].shape,               # H 4096, 32 heads x 128, F 11008, V 32000
    "13b": WORKLOADS["c2"].shape,              # H 5120, 40 heads x 128, F 13824, V 32000
    "8b_gqa": WORKLOADS["c4"].shape,           # H 4096, 32 query / 8 kv heads x 128, F 14336, V 128256
}


def _draft(name, shape, batch, kv_lo, kv_hi, n_new, k, topk, inputs="hidden", ragged=False, sample=False, probs=False):
    case = {"kind": "draft", "shape": shape, "batch": batch, "kv_lo": kv_lo, "kv_hi": kv_hi, "n_new": n_new, "k": k,
            "topk": topk, "inputs": inputs, "ragged": ragged, "sample": sample, "probs": probs}
    return dict(case, name=name) if name else case


def _verify(name, vocab, batch, fanout, rows, topk, agreement=0.7):
    case = {"kind": "verify", "vocab": vocab, "batch": batch, "fanout": fanout, "rows": rows, "topk": topk, "agreement": agreement}
    return dict(case, name=name) if name else case


def _train(name, dtype, seqs, tokens, k, n_heads, n_kv_heads, head_dim):
    case = {"kind": "train", "dtype": dtype, "seqs": seqs, "tokens": tokens, "k": k, "n_heads": n_heads,
            "n_kv_heads": n_kv_heads, "head_dim": head_dim}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest step: nothing but latency (the float32 drafter of the correctness workload)
        _draft("draft_tiny_f32", "tiny", 1, 64, 64, 1, 4, 4),
        # one sequence, one accepted token: the ordinary decode step of a 7B target's drafter
        _draft("draft_7b", "7b", 1, 512, 512, 1, 5, 8),
        # feature-fusion input (the drafter reads the target's features and the tokens), several accepted tokens
        _draft("draft_13b_features", "13b", 1, 1024, 1024, 4, 5, 8, inputs="features"),
        # a small serving batch that samples: token ids in, different accepted lengths, one draw per row at T = 1,
        # and the full distributions that the acceptance walk needs
        _draft("draft_7b_batch4_sampled", "7b", 4, 70, 1337, 3, 4, 8, inputs="tokens", ragged=True, sample=True, probs=True),
        # a larger ragged batch
        _draft("draft_7b_batch8", "7b", 8, 128, 2048, 1, 5, 8),
        # grouped-query attention, a large vocabulary and a long cache: the largest step of one sequence
        _draft("draft_8b_gqa_4k", "8b_gqa", 1, 4096, 4096, 1, 8, 8),
        # a round's tree and walk for one sequence, the 61-node tree over six draft rows
        _verify("verify_32k", 32000, 1, "4,2,2,1,1", 6, 8),
        # the same for a batch with a large vocabulary
        _verify("verify_128k_batch8", 128256, 8, "4,2,2,1,1", 9, 8),
        # training: one sequence at the context length the 7B drafter is trained with
        _train("train_2048", "bf16", 1, 2048, 4, 32, 32, 128),
        # a batch of sequences, grouped-query attention, nine rows per group
        _train("train_batch4_gqa", "bf16", 4, 1024, 8, 32, 8, 128),
        # one short conversation, odd length, six rows per group
        _train("train_short", "bf16", 1, 203, 5, 40, 40, 128),
        # a small float32 drafter
        _train("train_f32", "f32", 2, 300, 3, 8, 8, 64),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("draft", "verify", "train"), (5, 2, 4))[0]
    if kind == "draft":
        shape = rng.choice(("tiny", "small", "small_f32", "7b", "7b", "13b", "8b_gqa"))
        s = SHAPES[shape]
        group = s.n_heads // s.n_kv_heads
        k = rng.randint(1, 8)
        n_new = rng.randint(1, min(k + 1, 64 // group - k))
        batch = min(_log_int(rng, 1, 10), 64 // (n_new + k))
        kv_hi = _log_int(rng, 16, 4096 if batch == 1 else 2048)
        kv_lo = kv_hi if batch == 1 else rng.randint(1, kv_hi)
        sample = rng.random() < 0.3
        inputs = rng.choice(("hidden", "tokens", "features"))
        return _draft(None, shape, batch, kv_lo, kv_hi, n_new, k, rng.choice((1, 4, 8, 8, 10, 16)), inputs=inputs,
                      ragged=batch > 1 and n_new > 1 and rng.random() < 0.5, sample=sample, probs=sample and rng.random() < 0.5)
    if kind == "verify":
        fanout = rng.choice(("4,2,2,1,1", "3,2,1,1,1,1,1,1", "2,2,2,2", "1,1,1,1,1", "8,3,1", "5,1,1"))
        vocab = rng.choice((32000, 128256, _log_int(rng, 1000, 131072), 4 * _log_int(rng, 250, 32768)))
        return _verify(None, vocab, _log_int(rng, 1, max(1, min(16, 1100000 // vocab))), fanout, len(fanout.split(",")) + rng.randint(0, 1),
                       8, rng.choice((0.4, 0.7, 0.9)))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    head_dim = rng.choice((64, 128, 128)) if dtype == "bf16" else 64
    n_heads, n_kv_heads = rng.choice(((8, 8), (32, 32), (32, 8), (40, 40)) if head_dim == 128 else ((8, 8), (4, 4), (16, 4)))
    k = rng.randint(0, 10)
    tokens = _log_int(rng, 16, 2048 if dtype == "bf16" else 512)
    seqs = rng.randint(1, max(1, min(8, 2048 // tokens)))
    # (no more work than train_batch4_gqa)
    tokens = min(tokens, int(1024 * math.sqrt(4 * 9 * 32 / (seqs * (k + 1) * n_heads))))
    return _train(None, dtype, seqs, tokens, k, n_heads, n_kv_heads, head_dim)


# ------------------------------------------------------------------------------------------ states
def _kv_lens(case):
    """Lengths spread evenly over [kv_lo, kv_hi], not in order."""
    n, lo, hi = case["batch"], case["kv_lo"], case["kv_hi"]
    order = sorted(range(n), key=lambda i: (i * 5 + 3) % 11)
    return [hi if n == 1 else lo + (hi - lo) * i // (n - 1) for i in order]


def _accepted(case):
    """Accepted tokens per sequence: all n_new, or 1 .. n_new in turn."""
    n = case["n_new"]
    return [1 + (2 * b + 1) % n if case["ragged"] else n for b in range(case["batch"])]


def _torch_dtype(dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float32


class _DraftState:
    def __init__(self, case, seed):
        s = SHAPES[case["shape"]]
        g = torch.Generator(device=DEVICE).manual_seed(seed)
        dt = _torch_dtype(s.dtype)
        batch, n_new, k, topk = case["batch"], case["n_new"], case["k"], case["topk"]

        def normal(*shape, std=0.02, mean=0.0):
            return torch.empty(shape, dtype=dt, device=DEVICE).normal_(mean, std, generator=g)

        H = s.hidden
        w = {"g_in": normal(H, mean=1.0), "wq": normal(s.q_dim, H), "wk": normal(s.kv_dim, H), "wv": normal(s.kv_dim, H),
             "wo": normal(H, s.q_dim), "g_post": normal(H, mean=1.0), "w_gate": normal(s.ffn, H), "w_up": normal(s.ffn, H),
             "w_down": normal(H, s.ffn), "g_final": normal(H, mean=1.0), "w_lm": normal(s.vocab, H), "mask_emb": normal(k, H, std=1.0)}
        fused = case["inputs"] == "features"
        if case["inputs"] != "hidden":
            w["embed"] = normal(s.vocab, H, std=1.0)
        if fused:
            w["w_fc"] = normal(H, 2 * H, std=1.0 / math.sqrt(2.0 * H))
            w["b_fc"] = normal(H)
        self.weights_dev = w
        self.weights = B.ps_draft_weights()
        for n, t in w.items():
            setattr(self.weights, n, t.data_ptr())

        lens, acc = _kv_lens(case), _accepted(case)
        self.config = B.make_config(s, batch, n_new, max(lens) + n_new + k, topk, k_max=k, input_fc=fused)
        nbytes = B.ps_draft_workspace_bytes(self.config)
        self.workspace = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEVICE)
        st, self.ctx = B.ps_draft_init(self.config, self.weights, (self.workspace.data_ptr() + 255) & ~255, nbytes, _stream())
        if st != B.PS_OK:
            raise B.PsDraftError(st)

        off = [0]
        for n in lens:
            off.append(off[-1] + n + n_new + k)
        rows = k + 1
        self.k_cache, self.v_cache = normal(off[-1], s.n_kv_heads, s.head_dim), normal(off[-1], s.n_kv_heads, s.head_dim)
        self.out = {"top_ids": torch.empty((batch, rows, topk), dtype=torch.int32, device=DEVICE),
                    "top_p": torch.empty((batch, rows, topk), device=DEVICE), "lse": torch.empty((batch, rows), device=DEVICE)}
        if case["probs"]:
            self.out["probs"] = torch.empty((batch, rows, s.vocab), device=DEVICE)
        if case["sample"]:
            self.out["sample_ids"] = torch.empty((batch, rows), dtype=torch.int32, device=DEVICE)
            self.out["sample_p"] = torch.empty((batch, rows), device=DEVICE)
        a = self.args = B.ps_draft_step_args()
        a.batch, a.n_new, a.k, a.topk = batch, n_new, k, topk
        a.k_cache, a.v_cache = self.k_cache.data_ptr(), self.v_cache.data_ptr()
        self.host = ((ctypes.c_int64 * (batch + 1))(*off), (ctypes.c_int32 * batch)(*lens), (ctypes.c_int32 * batch)(*acc))
        a.kv_offsets = ctypes.cast(self.host[0], ctypes.POINTER(ctypes.c_int64))
        a.kv_len = ctypes.cast(self.host[1], ctypes.POINTER(ctypes.c_int32))
        if case["ragged"]:
            a.n_new_seq = ctypes.cast(self.host[2], ctypes.POINTER(ctypes.c_int32))
        if case["inputs"] == "hidden":
            self.x = normal(batch, n_new, H, std=1.0)
            a.x = self.x.data_ptr()
        else:
            self.token_ids = torch.randint(0, s.vocab, (batch, n_new), generator=g, device=DEVICE, dtype=torch.int32)
            a.token_ids = self.token_ids.data_ptr()
        if fused:
            self.features = normal(batch, n_new, H, std=1.0)
            a.features = self.features.data_ptr()
        if case["sample"]:
            a.temperature, a.sample_seed = 1.0, seed
        for n, t in self.out.items():
            setattr(a, n, t.data_ptr())

    def run(self):
        st = B.ps_draft_step(self.ctx, self.args, _stream())
        if st != B.PS_OK:
            raise B.PsDraftError(st)
        # (the step appends its rows to the caller's cache: updated state)
        return dict(self.out, k_cache=self.k_cache, v_cache=self.v_cache)

    def __del__(self):
        if getattr(self, "ctx", None) and B is not None:   # (None while the interpreter ends)
            B.ps_draft_free(self.ctx)
            self.ctx = None


class _VerifyState:
    def __init__(self, case, seed):
        g = torch.Generator(device=DEVICE).manual_seed(seed)
        V, batch, rows, topk, agree = case["vocab"], case["batch"], case["rows"], case["topk"], case["agreement"]
        parent, rank = draft_tree([int(f) for f in case["fanout"].split(",")])
        n = len(parent)
        depth = [0] * n
        for i in range(1, n):
            depth[i] = depth[parent[i]] + 1
        self.tree = VF.make_tree(parent, rank)

        def peaked(*shape):   # like a language model's next-token distributions
            return torch.softmax(4.0 * torch.randn(shape, generator=g, device=DEVICE), dim=-1)

        # the target after a node of depth t agrees with draft row t to a share of `agreement`
        self.q = peaked(batch, rows, V)
        self.p = peaked(batch, n, V)
        for i in range(n):
            if depth[i] < rows:
                self.p[:, i].mul_(1.0 - agree).add_(self.q[:, depth[i]], alpha=agree)
        self.top_ids = torch.topk(self.q, topk, dim=-1).indices.to(torch.int32).contiguous()
        self.r = torch.rand((batch, n), generator=g, device=DEVICE).clamp_(max=1.0 - 2.0 ** -24)
        i32 = dict(dtype=torch.int32, device=DEVICE)
        self.tokens, self.n_acc = torch.zeros((batch, n), **i32), torch.zeros((batch,), **i32)
        self.path, self.out_tokens = torch.zeros((batch, rows), **i32), torch.zeros((batch, rows + 1), **i32)
        a = self.args = VF.ps_verify_args()
        a.batch, a.rows, a.vocab = batch, rows, V
        a.tokens, a.q, a.p, a.r = self.tokens.data_ptr(), self.q.data_ptr(), self.p.data_ptr(), self.r.data_ptr()
        a.n_accepted, a.path, a.out_tokens = self.n_acc.data_ptr(), self.path.data_ptr(), self.out_tokens.data_ptr()
        nbytes = VF.ps_verify_workspace_bytes(batch, V)
        if nbytes:
            self.workspace = torch.zeros(nbytes + 256, dtype=torch.uint8, device=DEVICE)
            a.workspace, a.workspace_bytes = (self.workspace.data_ptr() + 255) & ~255, nbytes
        self.shape = (batch, rows, topk)

    def run(self):
        batch, rows, topk = self.shape
        stream = _stream()
        st = VF.ps_tree_tokens(self.tree, batch, rows, topk, self.top_ids.data_ptr(), self.tokens.data_ptr(), stream)
        st = st or VF.ps_verify_walk(self.tree, self.args, stream)
        if st != B.PS_OK:
            raise B.PsDraftError(st)
        return {"tokens": self.tokens, "n_accepted": self.n_acc, "path": self.path, "out_tokens": self.out_tokens}


class _TrainState:
    def __init__(self, case, seed):
        g = torch.Generator(device=DEVICE).manual_seed(seed)
        c = case
        dt, rows, d = _torch_dtype(c["dtype"]), c["tokens"] * (c["k"] + 1), c["head_dim"]

        def normal(heads):
            return torch.empty((c["seqs"], rows, heads, d), dtype=dt, device=DEVICE).normal_(0.0, 1.0, generator=g)

        self.q, self.k, self.v = normal(c["n_heads"]), normal(c["n_kv_heads"]), normal(c["n_kv_heads"])
        self.out = torch.empty((c["seqs"], rows, c["n_heads"], d), dtype=torch.float32, device=DEVICE)
        a = self.args = TR.make_args(c["seqs"], c["tokens"], c["k"], c["n_heads"], c["n_kv_heads"], d, c["dtype"], 10000.0)
        nbytes = TR.ps_group_attention_workspace_bytes(a)
        self.workspace = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEVICE)
        a.q, a.k_, a.v, a.out = self.q.data_ptr(), self.k.data_ptr(), self.v.data_ptr(), self.out.data_ptr()
        a.workspace, a.workspace_bytes = (self.workspace.data_ptr() + 255) & ~255, nbytes

    def run(self):
        st = TR.ps_group_attention(self.args, _stream())
        if st != B.PS_OK:
            raise B.PsDraftError(st)
        return self.out


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def prepare(case, seed):
    return {"draft": _DraftState, "verify": _VerifyState, "train": _TrainState}[case["kind"]](case, seed)


def run(state):
    return state.run()


# ------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    if case["kind"] == "draft":
        s = SHAPES[case["shape"]]
        esz = 2 if s.dtype == "bf16" else 4
        k, lens, acc = case["k"], _kv_lens(case), _accepted(case)
        H, rows, outs = s.hidden, sum(acc) + case["batch"] * k, case["batch"] * (k + 1)
        layer = s.layer_params()
        head = s.vocab * H
        fc = 2 * H * H if case["inputs"] == "features" else 0
        pairs = sum((n + (a + k + 1) / 2) * (a + k) for n, a in zip(lens, acc))
        nbytes = esz * (layer + head + fc + 2 * s.kv_dim * (sum(lens) + rows) + sum(acc) * H + k * H)
        nbytes += outs * (4 + 8 * case["topk"]) + (4 * outs * s.vocab if case["probs"] else 0)
        return {"bytes": nbytes, "flops": 2.0 * (layer * rows + head * outs + fc * sum(acc)) + 4.0 * s.q_dim * pairs}
    if case["kind"] == "verify":
        # a rejection (there is one in nearly every walk) reads a row of the target and one of the drafter
        return {"bytes": 8.0 * case["batch"] * case["vocab"], "flops": 4.0 * case["batch"] * case["vocab"]}
    c = case
    esz = 2 if c["dtype"] == "bf16" else 4
    T, k, d = c["tokens"], c["k"], c["head_dim"]
    rows = T * (k + 1)
    pairs = (k + 1) * T * (T + 1) // 2 + T * k * (k + 1) // 2
    return {"bytes": c["seqs"] * rows * d * (esz * (c["n_heads"] + 2 * c["n_kv_heads"]) + 4 * c["n_heads"]),
            "flops": 4.0 * d * pairs * c["n_heads"] * c["seqs"]}


def tolerance(case):
    """About four times what two correct orders of the same sums differ by (other K splits of the draft step's
    products; the training attention against float64).  draft: probabilities by 1e-5; where a new K/V element lies on a
    rounding boundary of its bf16 cache it moves by one unit in the last place (8e-3 of its value), and what depends on
    it by up to 6e-5; token ids may differ where two logits tie to within that.  verify: decisions are taken in float64.
    train: 2.4e-7 in float32; in bf16 2e-5, single values by 1.4e-3, where a rotated key moves by one unit."""
    if case["kind"] == "verify":
        return "exact"
    if case["kind"] == "draft":
        return {"rel": 1e-5, "max": 2e-4, "differ": 0.01} if SHAPES[case["shape"]].dtype == "f32" else {"rel": 3e-4, "max": 3e-2, "differ": 0.01}
    return {"rel": 2e-6, "max": 3e-5} if case["dtype"] == "f32" else {"rel": 1e-4, "max": 1e-2}
