"""Performance cases of the candidate-evaluation path: what a program that uses this framework has it do, through the
public entry points (the calls of `binding`, the driver objects of `runner`).

A case is a dict of plain values.  `kind` names the call:

    step     fp32 probe linear + scoring of one small layer and head: the whole path at its smallest
    linear   one bf16 probe linear (plain, ReLU, gated SiLU; with and without bank, bias, foreground rows)
    score    bf16 scoring against an LM head, every token or only the last tokens of every sequence
    attn     causal attention over the packed sequences
    joins    residual sum + norm, then per-head q/k norm + rotary embedding: the memory-bound calls of a block
    update   estimate + lazy bank update of the probed layers of a model: what ends a step
    model    the teacher-forced scoring pass of a small whole model (runner.DeviceModel)

Batches are packed the way the framework's own workloads are: every example appears as a (+, -) pair of sequences with
the same rows, directions are dealt to the examples in turn, foreground sequences may be mixed in, and then the order
is shuffled.  Inputs have the distributions of those workloads: rows N(0, 1), weights N(0, 1/fan-in), bank N(0, 1e-4).
"""
import math
import random
from collections import namedtuple

import numpy as np
import torch

from paper_2605_28760_amd import binding as zb
from paper_2605_28760_amd import workloads as wl
from paper_2605_28760_amd.runner import DeviceBatch, DeviceModel, DeviceWorkload

EPS = 1e-3
LR = 1e-6


# ---- the cases ------------------------------------------------------------------------------------------------------

def listed():
    return [
        # the fp32 configuration: one 256 x 256 linear and a 512-row head, 8 examples under the candidates +, -, centre:
        # a smoke run or a unit-sized experiment, where launches and latency count
        dict(name="step_f32_tiny", kind="step", d=256, vocab=512, n_ex=8, lo=32, hi=32, n_dirs=1, centre=True, n_fg=0,
             lens=1, r=4, R=0),
        # one example under its two candidates (batch size 1, a prompt of a sentence) through a Qwen3-8B attention
        # output projection: the smallest bf16 call, weights streamed for a few rows
        dict(name="linear_one_prompt", kind="linear", m=4096, n=4096, n_ex=1, lo=48, hi=48, n_dirs=1, n_fg=0, lens=2,
             r=16, R=128, act=0, bias=False, f32_out=False),
        # batch size 16 of short classification prompts through OPT-13B's fc1 (bias, ReLU)
        dict(name="linear_b16_fc1", kind="linear", m=20480, n=5120, n_ex=16, lo=16, hi=64, n_dirs=1, n_fg=0, lens=3,
             r=8, R=64, act=1, bias=True, f32_out=False),
        # batch size 64 of 128-token examples through OPT-13B's fc2: the scoring benchmark's shape
        dict(name="linear_b64_fc2", kind="linear", m=5120, n=20480, n_ex=64, lo=128, hi=128, n_dirs=1, n_fg=0, lens=4,
             r=8, R=64, act=0, bias=True, f32_out=False),
        # co-serving batch on Qwen3-8B: ragged probe pairs of 24 directions mixed with foreground sequences through the
        # fused gate/up projection with the gated activation: the largest call
        dict(name="linear_mixed_gate", kind="linear", m=24576, n=4096, n_ex=24, lo=64, hi=1024, n_dirs=24, n_fg=16,
             lens=5, r=16, R=128, act=2, bias=False, f32_out=False),
        # every token of a ragged batch scored against Qwen3-8B's 151936-row head
        dict(name="score_all_tokens", kind="score", vocab=151936, d=4096, n_ex=16, lo=16, hi=512, n_dirs=16, n_fg=0,
             lens=6, last=0),
        # classification: only the label token of every sequence of a batch of 64 pairs is scored, OPT's 50272-row head
        dict(name="score_label_token", kind="score", vocab=50272, d=5120, n_ex=64, lo=128, hi=128, n_dirs=1, n_fg=0,
             lens=7, last=1),
        # attention of a Qwen3-8B block (32 query heads over 8) on a ragged batch of prompts of up to 512 tokens
        dict(name="attn_ragged_gqa", kind="attn", heads=32, kv=8, n_ex=32, lo=16, hi=512, n_dirs=16, n_fg=0, lens=8),
        # attention of an OPT-13B block (40 heads) on documents of 2048 tokens, the model's context length
        dict(name="attn_long", kind="attn", heads=40, kv=40, n_ex=4, lo=2048, hi=2048, n_dirs=1, n_fg=0, lens=9),
        # the memory-bound calls around attention in a Qwen3-8B block on the same kind of ragged batch
        dict(name="joins_ragged", kind="joins", d=4096, norm=1, heads=32, kv=8, n_ex=32, lo=16, hi=512, n_dirs=16,
             n_fg=0, lens=10),
        # end of a step of an 8-direction run: estimate, then the update of 36 layers (12288 x 4096, rank 16)
        dict(name="update_36_layers", kind="update", layers=36, m=12288, n=4096, n_ex=8, lo=16, hi=16, n_dirs=8, n_fg=0,
             lens=11, r=16, R=128),
        # a whole small model of the Qwen3 form (two blocks, hidden 1024, 32000-row head) on batch size 16
        dict(name="model_small", kind="model", blocks=2, hidden=1024, heads=8, kv=4, ffn=3072, vocab=32000, n_ex=16,
             lo=16, hi=64, n_dirs=4, n_fg=2, lens=12, r=8, R=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch_of(rng, rows_lo, rows_hi, len_hi, dirs_hi, fg=True):
    """Fields of a batch of about `rows` rows: log-uniform in rows and in the longest sequence."""
    rows = _log(rng, rows_lo, rows_hi)
    hi = min(_log(rng, 16, len_hi), max(rows // 2, 8))
    lo = hi if rng.random() < 0.3 else max(1, hi // rng.choice([2, 4, 16, 32]))
    n_ex = max(1, round(rows / (lo + hi)))
    return dict(n_ex=n_ex, lo=lo, hi=hi, n_dirs=min(n_ex, _log(rng, 1, dirs_hi)),
                n_fg=rng.randint(0, n_ex) if fg and rng.random() < 0.4 else 0, lens=rng.randrange(1 << 30))


def draw(rng):
    while True:
        case = _draw(rng)
        if work(case)["flops"] <= 8e12:   # no dearer than the listed ones
            return case


def _draw(rng):
    kind = rng.choice(["step", "linear", "linear", "linear", "score", "score", "attn", "attn", "joins", "update",
                       "model"])
    if kind == "step":
        c = _batch_of(rng, 64, 4096, 256, 4)
        c.update(d=rng.randint(32, 640), vocab=_log(rng, 100, 5000), centre=rng.random() < 0.5, r=rng.choice([1, 4, 8, 10]),
                 R=rng.choice([0, 0, 8, 33]))
    elif kind == "linear":
        c = _batch_of(rng, 32, 16384, 1024, 24)
        m, n, act = rng.choice([(4096, 4096, 0), (6144, 4096, 0), (5120, 5120, 0), (15360, 5120, 0), (20480, 5120, 1),
                                (5120, 20480, 0), (4096, 12288, 0), (24576, 4096, 2), (0, 0, 0), (0, 0, 1), (0, 0, 2)])
        if m == 0:   # widths of no particular model
            m, n = 8 * _log(rng, 32, 2000), 64 * _log(rng, 6, 200)
            m = (m + 15) // 16 * 16 if act == 2 else m
        c.update(m=m, n=n, act=act, r=rng.choice([4, 8, 16, 16, 33, 64]), R=rng.choice([0, 16, 64, 64, 128, 200]),
                 bias=rng.random() < 0.5, f32_out=rng.random() < 0.15)
    elif kind == "score":
        c = _batch_of(rng, 64, 12000, 1024, 24)
        vocab, d = rng.choice([(50272, 5120), (151936, 4096), (32000, 4096), (0, 0)])
        if vocab == 0:
            vocab, d = _log(rng, 1000, 130000), 64 * _log(rng, 8, 80)
        c.update(vocab=vocab, d=d, last=rng.choice([0, 0, 1, 4, 16]))
    elif kind == "attn":
        c = _batch_of(rng, 64, 16384, 4096, 8)
        heads, kv = rng.choice([(40, 40), (32, 8), (16, 16), (8, 4), (12, 1)])
        c.update(heads=heads, kv=kv)
    elif kind == "joins":
        c = _batch_of(rng, 64, 32768, 1024, 24)
        heads, kv = rng.choice([(40, 40), (32, 8), (8, 4), (5, 1)])
        c.update(heads=heads, kv=kv, d=rng.choice([4096, 5120, 1024, 8 * _log(rng, 64, 900)]), norm=rng.randint(0, 1))
    elif kind == "update":
        c = _batch_of(rng, 64, 512, 16, 16, fg=False)
        c.update(layers=rng.randint(1, 40), m=8 * _log(rng, 128, 2560), n=8 * _log(rng, 128, 1536), r=rng.choice([4, 8, 16, 6]))
        c["R"] = c["n_dirs"] * c["r"] + rng.choice([0, 0, 16])
    else:
        c = _batch_of(rng, 64, 2048, 256, 8)
        heads, kv = rng.choice([(8, 8), (8, 4), (4, 1)])
        c.update(blocks=rng.randint(1, 3), hidden=rng.choice([512, 1024, 1280]), heads=heads, kv=kv,
                 ffn=rng.choice([1536, 3072, 4096]), vocab=rng.choice([8192, 32000, 50272]), r=rng.choice([4, 8, 16]),
                 R=rng.choice([16, 32, 64]))
    c["kind"] = kind
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------------

Packed = namedtuple("Packed", "cu cand cand_dir cand_sign ex lens ex_off")


def _packed(case):
    """The packed batch of a case: sequence bounds, candidate of every sequence, candidate table, example of every
    sequence, and where an example's rows start in the list of distinct rows."""
    rnd = random.Random(case["lens"])
    K = case["n_dirs"]
    per = 3 if case.get("centre") else 2
    seqs, sizes = [], []
    for e in range(case["n_ex"]):
        sizes.append(rnd.randint(case["lo"], case["hi"]))
        k = e % K
        seqs += [(e, 2 * k), (e, 2 * k + 1)] + ([(e, 2 * K)] if per == 3 else [])
    for f in range(case["n_fg"]):
        sizes.append(rnd.randint(case["lo"], case["hi"]))
        seqs.append((case["n_ex"] + f, -1))
    if case["n_fg"]:
        rnd.shuffle(seqs)
    cand_dir = np.repeat(np.arange(K, dtype=np.int32), 2)
    cand_sign = np.tile(np.array([1, -1], np.float32), K)
    if per == 3:
        cand_dir, cand_sign = np.append(cand_dir, np.int32(-1)), np.append(cand_sign, np.float32(0))
    ex = np.array([s[0] for s in seqs], np.int64)
    lens = np.array(sizes, np.int64)[ex]
    cu = np.zeros(len(seqs) + 1, np.int32)
    cu[1:] = np.cumsum(lens)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return Packed(cu, np.array([s[1] for s in seqs], np.int32), cand_dir, cand_sign, ex, lens, off)


def _rows_of(pk):
    """Index of every packed row into the list of distinct rows (both sequences of a pair hold the same rows)."""
    return np.concatenate([np.arange(pk.ex_off[e], pk.ex_off[e] + n) for e, n in zip(pk.ex, pk.lens)])


def _seeds(case, seed):
    return (np.uint64(0x5EED0000) + np.uint64(seed % (1 << 31)) * np.uint64(1000) + np.arange(case["n_dirs"], dtype=np.uint64))


class _Source:
    """Seeded random tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, shape, std=1.0, dtype=torch.float32):
        x = torch.randn(shape, device="cuda", dtype=torch.float32, generator=self.g)
        return x.mul_(std).to(dtype)

    def packed_rows(self, pk, width, dtype):
        base = self.normal((int(pk.ex_off[-1]), width), 1.0, dtype)
        return base[torch.from_numpy(_rows_of(pk)).cuda()].contiguous()

    def targets(self, pk, vocab, last=0):
        base = torch.randint(0, vocab, (int(pk.ex_off[-1]),), device="cuda", dtype=torch.int32, generator=self.g)
        t = base[torch.from_numpy(_rows_of(pk)).cuda()].contiguous()
        if last:   # only the last `last` rows of a sequence carry a target
            left = np.concatenate([np.arange(n, 0, -1) for n in pk.lens])
            t[torch.from_numpy(left > last).cuda()] = -1
        return t


def _batch(case, seed, pk):
    return DeviceBatch(pk.cu, pk.cand, pk.cand_dir, pk.cand_sign, _seeds(case, seed), "cuda")


def _inputs(case, seed):
    """Everything random of a case, as tensors on the GPU."""
    k, pk, s = case["kind"], _packed(case), _Source(seed)
    T = int(pk.cu[-1])
    x = {"pk": pk}
    if k == "step":
        d, f32 = case["d"], torch.float32
        x.update(X=s.packed_rows(pk, d, f32), W=s.normal((d, d), d ** -0.5), head=s.normal((case["vocab"], d), d ** -0.5),
                 P=s.normal((d, case["R"]), 1e-2), Vb=s.normal((d, case["R"]), 1e-2), targets=s.targets(pk, case["vocab"]))
    elif k == "linear":
        m, n, bf = case["m"], case["n"], torch.bfloat16
        x.update(X=s.packed_rows(pk, n, bf), W=s.normal((m, n), n ** -0.5, bf), P=s.normal((m, case["R"]), 1e-2),
                 Vb=s.normal((n, case["R"]), 1e-2), bias=s.normal((m,), 0.1) if case["bias"] else None)
    elif k == "score":
        d, bf = case["d"], torch.bfloat16
        x.update(H=s.packed_rows(pk, d, bf), head=s.normal((case["vocab"], d), d ** -0.5, bf),
                 targets=s.targets(pk, case["vocab"], case["last"]))
    elif k in ("attn", "joins"):
        bf = torch.bfloat16
        x["qkv"] = s.packed_rows(pk, (case["heads"] + 2 * case["kv"]) * 128, bf)
        if k == "joins":
            d = case["d"]
            x.update(X=s.packed_rows(pk, d, bf), res=s.normal((T, d), 1.0, bf), gamma=1 + s.normal((d,), 0.1),
                     beta=s.normal((d,), 0.1) if case["norm"] == 0 else None, gq=1 + s.normal((128,), 0.1),
                     gk=1 + s.normal((128,), 0.1))
    elif k == "update":
        C = 2 * case["n_dirs"]
        x.update(P=[s.normal((case["m"], case["R"]), 1e-2) for _ in range(case["layers"])],
                 Vb=[s.normal((case["n"], case["R"]), 1e-2) for _ in range(case["layers"])],
                 cand_sum=(s.normal((C,), 1.0) + 40.0) * 16, cand_cnt=torch.full((C,), 16, device="cuda", dtype=torch.int32))
    return x


def _model_workload(case, seed):
    pk = _packed(case)
    batch = (pk.cu, pk.cand, pk.cand_dir, pk.cand_sign, pk.ex, pk.lens)
    return wl.decoder_model("model", seed % (1 << 31), "bf16", case["blocks"], case["hidden"], case["heads"], case["kv"],
                            128, case["ffn"], case["vocab"], 1, False, case["r"], EPS, case["R"], batch, qwen=True)


# ---- one pass -------------------------------------------------------------------------------------------------------

class State:
    pass


def prepare(case, seed):
    st = State()
    st.case = case
    if case["kind"] == "model":
        st.model = DeviceModel(DeviceWorkload(_model_workload(case, seed), "cuda"))
        return st
    x = _inputs(case, seed)
    pk = x.pop("pk")
    st.b = _batch(case, seed, pk)
    for name, v in x.items():
        setattr(st, name, v)
    T, S, C, K = st.b.T, st.b.S, st.b.C, st.b.K
    empty = lambda shape, dt=torch.float32: torch.empty(shape, device="cuda", dtype=dt)
    kind, ws = case["kind"], 256
    if kind in ("step", "linear"):
        m, n = (case["d"], case["d"]) if kind == "step" else (case["m"], case["n"])
        st.bank = zb.make_bank(case["R"], case["R"], st.P, st.Vb) if case["R"] else None
        dt = zb.ZO_F32 if kind == "step" else zb.ZO_BF16
        ws = max(ws, zb.zo_probe_linear_workspace_bytes(T, S, K, m, n, case["r"], case["R"], dt))
        if kind == "step":
            st.Y = empty((T, m))
        else:
            st.Y = empty((T, m // 2 if case["act"] == 2 else m), torch.float32 if case["f32_out"] else torch.bfloat16)
    if kind in ("step", "score"):
        dt = zb.ZO_F32 if kind == "step" else zb.ZO_BF16
        ws = max(ws, zb.zo_score_workspace_bytes(T, S, case["vocab"], case["d"], dt))
        st.tok_nll, st.seq_nll, st.cand_sum = empty(T), empty(S), empty(C)
        st.cand_cnt = empty(C, torch.int32)
    if kind == "attn":
        st.O = empty((T, case["heads"] * 128), torch.bfloat16)
    if kind == "joins":
        st.hsum, st.y = torch.empty_like(st.X), torch.empty_like(st.X)
    if kind == "update":
        st.cand_loss, st.proj_grad = empty(C), empty(K)
        banks = [zb.make_bank(case["R"], case["R"], P, Vb) for P, Vb in zip(st.P, st.Vb)]
        st.layers = zb.make_layer_banks([(k, case["m"], case["n"], 2 * i) for i, k in enumerate(banks)])
        st.col0 = np.arange(K, dtype=np.int32) * case["r"]
    st.ws_bytes = ws
    st.ws = torch.empty(ws, device="cuda", dtype=torch.uint8)
    return st


def run(st):
    c = st.case
    kind = c["kind"]
    if kind == "model":
        d = st.model.d
        final = st.model.forward()
        return {"final": final, "tok_nll": d.tok_nll, "seq_nll": d.seq_nll, "cand_sum": d.cand_sum, "cand_cnt": d.cand_cnt}
    b = st.b
    if kind == "linear":
        zb.zo_probe_linear(b.struct, st.X, c["n"], st.W, c["n"], st.bias, c["m"], c["n"], zb.ZO_BF16, c["r"], EPS, 2,
                           st.bank, c["act"], st.Y, st.Y.stride(0), zb.ZO_F32 if c["f32_out"] else zb.ZO_BF16, st.ws,
                           st.ws_bytes)
        return {"Y": st.Y}
    if kind == "step":
        d = c["d"]
        zb.zo_probe_linear(b.struct, st.X, d, st.W, d, None, d, d, zb.ZO_F32, c["r"], EPS, 2, st.bank, 0, st.Y, d,
                           zb.ZO_F32, st.ws, st.ws_bytes)
        zb.zo_score(b.struct, st.Y, d, st.head, d, c["vocab"], d, zb.ZO_F32, st.targets, st.tok_nll, st.seq_nll,
                    st.cand_sum, st.cand_cnt, st.ws, st.ws_bytes)
        return {"Y": st.Y, "tok_nll": st.tok_nll, "seq_nll": st.seq_nll, "cand_sum": st.cand_sum, "cand_cnt": st.cand_cnt}
    if kind == "score":
        zb.zo_score(b.struct, st.H, c["d"], st.head, c["d"], c["vocab"], c["d"], zb.ZO_BF16, st.targets, st.tok_nll,
                    st.seq_nll, st.cand_sum, st.cand_cnt, st.ws, st.ws_bytes)
        return {"tok_nll": st.tok_nll, "seq_nll": st.seq_nll, "cand_sum": st.cand_sum, "cand_cnt": st.cand_cnt}
    if kind == "update":
        zb.zo_estimate(b.struct, st.cand_sum, st.cand_cnt, EPS, 0, st.cand_loss, st.proj_grad)
        zb.zo_bank_update_multi(st.layers, c["r"], b.K, b.dir_seed, None, st.proj_grad, LR, None, st.col0, 0, zb.ZO_BF16)
        return {"cand_loss": st.cand_loss, "proj_grad": st.proj_grad, "P": list(st.P)}
    nq, nkv, ld = c["heads"] * 128, c["kv"] * 128, st.qkv.stride(0)
    q, k, v = st.qkv[:, :nq], st.qkv[:, nq:nq + nkv], st.qkv[:, nq + nkv:]
    if kind == "attn":
        zb.zo_attention(b.struct, q, ld, k, ld, v, ld, c["heads"], c["kv"], 128, 128 ** -0.5, zb.ZO_BF16, st.O, nq)
        return {"O": st.O}
    d = c["d"]
    zb.zo_add_norm(st.X, d, st.res, d, st.gamma, st.beta, c["norm"], 1e-6, b.T, d, zb.ZO_BF16, st.hsum, d, st.y, d)
    zb.zo_qk_norm_rope(b.struct, q, ld, k, ld, c["heads"], c["kv"], 128, st.gq, st.gk, 1e-6, 1e6, zb.ZO_BF16)
    return {"hsum": st.hsum, "y": st.y, "qkv": st.qkv}


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def _linear_work(T, pk, m, n, r, R, m_out, size, out_size):
    """Inputs once, outputs once; products of the base, and of the side state for the rows that have one."""
    rows = int(pk.lens[pk.cand >= 0].sum())
    return dict(bytes=(T * n + m * n) * size + T * m_out * out_size + (m + n) * R * 4,
                flops=2 * T * m * n + 2 * rows * (r + R) * (m + n))


def _score_work(pk, case, size):
    last = case.get("last", 0)
    n = int(np.minimum(pk.lens, last).sum()) if last else int(pk.cu[-1])
    return dict(bytes=(n + case["vocab"]) * case["d"] * size + 12 * int(pk.cu[-1]), flops=2 * n * case["vocab"] * case["d"])


def work(case):
    pk = _packed(case)
    T, kind = int(pk.cu[-1]), case["kind"]
    pairs = int((pk.lens * (pk.lens + 1) // 2).sum())   # (query, key) pairs of causal attention
    if kind == "step":
        d = case["d"]
        a, b = _linear_work(T, pk, d, d, case["r"], case["R"], d, 4, 4), _score_work(pk, case, 4)
        return dict(bytes=a["bytes"] + b["bytes"], flops=a["flops"] + b["flops"])
    if kind == "linear":
        return _linear_work(T, pk, case["m"], case["n"], case["r"], case["R"],
                            case["m"] // 2 if case["act"] == 2 else case["m"], 2, 4 if case["f32_out"] else 2)
    if kind == "score":
        return _score_work(pk, case, 2)
    if kind == "attn":
        return dict(bytes=T * (2 * case["heads"] + 2 * case["kv"]) * 256, flops=4 * 128 * case["heads"] * pairs)
    if kind == "joins":
        return dict(bytes=T * (8 * case["d"] + 4 * 128 * (case["heads"] + case["kv"])),
                    flops=T * (10 * case["d"] + 10 * 128 * (case["heads"] + case["kv"])))
    if kind == "update":
        n = case["layers"] * case["m"] * case["n_dirs"] * case["r"]
        return dict(bytes=8 * n, flops=2 * n)
    h, nq, nkv, f = case["hidden"], case["heads"] * 128, case["kv"] * 128, case["ffn"]
    total = dict(_score_work(pk, dict(vocab=case["vocab"], d=h), 2))
    for m, n, m_out in ((nq + 2 * nkv, h, nq + 2 * nkv), (h, nq, h), (2 * f, h, f), (h, f, h)):
        w = _linear_work(T, pk, m, n, case["r"], case["R"], m_out, 2, 2)
        total = {key: total[key] + case["blocks"] * w[key] for key in total}
    total["bytes"] += case["blocks"] * T * (2 * nq + 2 * nkv + 8 * h) * 2
    total["flops"] += case["blocks"] * 4 * 128 * case["heads"] * pairs
    return total


def tolerance(case):
    """About four times the error measured against 64 bits."""
    return {
        # fp32 throughout (3e-7)
        "step": {"rel": 2e-6, "max": 1e-4},
        # the output's rounding to bf16, the side terms' inside (1.8e-3)
        "linear": {"rel": 7e-3, "max": 6e-2},
        # fp32 sums of bf16 products, fp32 log-sum-exp (1e-7)
        "score": {"rel": 1e-6, "max": 4e-5},
        # weights rounded to bf16, output rounded to bf16 (2e-3)
        "attn": {"rel": 8e-3, "max": 8e-2},
        # stored sums and rows rounded to bf16 (1.8e-3)
        "joins": {"rel": 7e-3, "max": 4e-2},
        # factors are rounded to bf16: a normal next to a rounding boundary may fall either way (7e-7)
        "update": {"rel": 4e-6, "max": 1e-3},
        # bf16 storage, about eight roundings per block (5.5e-3)
        "model": {"rel": 2.2e-2, "max": 2e-1},
    }[case["kind"]]


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def _philox(seed, stream, blocks):
    """Philox4x32-10, counter (block, stream, 0), key = seed: four words per block, as int64 tensors."""
    M = 0xFFFFFFFF
    c = [blocks & M, blocks >> 32, torch.full_like(blocks, stream), torch.zeros_like(blocks)]
    k0, k1 = int(seed) & M, int(seed) >> 32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & M) ^ c[1] ^ k0, p1 & M, ((p0 >> 32) & M) ^ c[3] ^ k1, p0 & M]
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c


def _factor(seed, stream, rows, r, bf16):
    """[rows x r] standard normals by Box-Muller, rounded the way the factors are stored."""
    q = torch.arange((rows * r + 3) // 4, device="cuda", dtype=torch.int64)
    w = _philox(seed, stream, q)
    u = [(2 * (x >> 9) + 1).double() * 2.0 ** -24 for x in w]
    rho = [torch.sqrt(-2 * torch.log(u[0])), torch.sqrt(-2 * torch.log(u[2]))]
    ang = [2 * math.pi * u[1], 2 * math.pi * u[3]]
    z = torch.stack([rho[0] * torch.cos(ang[0]), rho[0] * torch.sin(ang[0]), rho[1] * torch.cos(ang[1]),
                     rho[1] * torch.sin(ang[1])], 1).reshape(-1)[:rows * r].reshape(rows, r)
    return z.float().to(torch.bfloat16).double() if bf16 else z


def _exact_linear(pk, seeds, X, W, bias, act, r, P, Vb, bf16, tensor_id):
    m, n = W.shape
    X = X.double()
    Y = X @ W.double().t()
    for k in range(len(seeds)):
        seqs = [s for s in range(len(pk.cand)) if pk.cand[s] >= 0 and pk.cand_dir[pk.cand[s]] == k]
        if not seqs:
            continue
        U, V = (_factor(seeds[k], t, rows, r, bf16) for t, rows in ((tensor_id, m), (tensor_id | 1, n)))
        for s in seqs:
            a, b = int(pk.cu[s]), int(pk.cu[s + 1])
            Y[a:b] += float(pk.cand_sign[pk.cand[s]]) * EPS * ((X[a:b] @ V) @ U.t())
    if P is not None and P.shape[1]:
        for s in range(len(pk.cand)):
            if pk.cand[s] >= 0:
                a, b = int(pk.cu[s]), int(pk.cu[s + 1])
                Y[a:b] += (X[a:b] @ Vb.double()) @ P.double().t()
    if bias is not None:
        Y += bias.double()
    if act == 1:
        Y.clamp_(min=0)
    elif act == 2:
        g, u = Y[:, 0::2], Y[:, 1::2]
        Y = g / (1 + torch.exp(-g)) * u
    return Y


def _exact_score(pk, H, head, targets):
    T = H.shape[0]
    tok = torch.zeros(T, device="cuda", dtype=torch.float64)
    rows = torch.nonzero(targets >= 0).flatten()
    Wd = head.double()
    for i in range(0, len(rows), 1024):
        r = rows[i:i + 1024]
        z = H[r].double() @ Wd.t()
        tok[r] = torch.logsumexp(z, 1) - z.gather(1, targets[r].long()[:, None])[:, 0]
    seq = torch.stack([tok[int(a):int(b)].sum() for a, b in zip(pk.cu[:-1], pk.cu[1:])])
    scored = torch.stack([(targets[int(a):int(b)] >= 0).sum() for a, b in zip(pk.cu[:-1], pk.cu[1:])])
    cand = torch.from_numpy(pk.cand).cuda()
    C = len(pk.cand_dir)
    zero = torch.zeros((), device="cuda", dtype=torch.float64)
    return {"tok_nll": tok, "seq_nll": seq,
            "cand_sum": torch.stack([torch.where(cand == c, seq, zero).sum() for c in range(C)]),
            "cand_cnt": torch.stack([scored[cand == c].sum() for c in range(C)]).to(torch.int32)}


def _exact_attention(pk, q, k, v, heads, kv):
    q, k, v = (x.double().reshape(x.shape[0], -1, 128) for x in (q, k, v))
    O = torch.empty_like(q)
    for a, b in zip(pk.cu[:-1], pk.cu[1:]):
        a, b = int(a), int(b)
        mask = torch.ones((b - a, b - a), device="cuda", dtype=torch.bool).tril()
        for h in range(heads):
            g = h // (heads // kv)
            s = (q[a:b, h] @ k[a:b, g].t()) * 128 ** -0.5
            O[a:b, h] = torch.softmax(s.masked_fill(~mask, -math.inf), 1) @ v[a:b, g]
    return O.reshape(O.shape[0], -1)


def _exact_norm(h, gamma, beta, kind):
    if kind == 0:
        y = (h - h.mean(1, keepdim=True)) / torch.sqrt(h.var(1, unbiased=False, keepdim=True) + 1e-6)
    else:
        y = h / torch.sqrt((h * h).mean(1, keepdim=True) + 1e-6)
    y = y * gamma.double()
    return y + beta.double() if beta is not None else y


def _exact_rope(pk, x, gamma):
    """Per-head RMS norm and rotary embedding of x [T x heads*128]."""
    x = x.double().reshape(x.shape[0], -1, 128)
    x = x / torch.sqrt((x * x).mean(2, keepdim=True) + 1e-6) * gamma.double()
    pos = torch.from_numpy(np.concatenate([np.arange(n) for n in pk.lens])).cuda().double()
    ang = pos[:, None] * (1e6 ** (-torch.arange(64, device="cuda", dtype=torch.float64) / 64))[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = x[..., :64], x[..., 64:]
    return torch.cat([a * c - b * s, b * c + a * s], 2).reshape(x.shape[0], -1)


def _exact_model(case, seed):
    w, pk = _model_workload(case, seed), _packed(case)
    up = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    nq, nkv = case["heads"] * 128, case["kv"] * 128

    def linear(layer, x):
        return _exact_linear(pk, w.dir_seed, x, up(layer.W), None, layer.act, case["r"], up(layer.P), up(layer.Vb), True,
                             layer.tensor_id)

    x = up(w.X).double()
    for blk in w.meta["blocks"]:
        qkv = linear(blk.qkv, _exact_norm(x, up(blk.g1), None, 1))
        q, k = _exact_rope(pk, qkv[:, :nq], up(blk.gq)), _exact_rope(pk, qkv[:, nq:nq + nkv], up(blk.gk))
        x = x + linear(blk.o, _exact_attention(pk, q, k, qkv[:, nq + nkv:], case["heads"], case["kv"]))
        x = x + linear(blk.fc2, linear(blk.fc1, _exact_norm(x, up(blk.g2), None, 1)))
    final = _exact_norm(x, up(w.meta["final_norm"][0]), None, 1)
    return {"final": final, **_exact_score(pk, final, up(w.head), up(w.targets))}


def exact(case, seed):
    kind = case["kind"]
    if kind == "model":
        return _exact_model(case, seed)
    x = _inputs(case, seed)
    pk, seeds = x["pk"], _seeds(case, seed)
    if kind == "linear":
        return {"Y": _exact_linear(pk, seeds, x["X"], x["W"], x["bias"], case["act"], case["r"], x["P"], x["Vb"], True, 2)}
    if kind == "step":
        Y = _exact_linear(pk, seeds, x["X"], x["W"], None, 0, case["r"], x["P"], x["Vb"], False, 2)
        return {"Y": Y, **_exact_score(pk, Y, x["head"], x["targets"])}
    if kind == "score":
        return _exact_score(pk, x["H"], x["head"], x["targets"])
    if kind == "update":
        loss = x["cand_sum"].double() / x["cand_cnt"].double()
        grad = (loss[0::2] - loss[1::2]) / (2 * EPS)
        r = case["r"]
        out = []
        for i, P in enumerate(x["P"]):
            P = P.double()
            for k in range(case["n_dirs"]):
                P[:, k * r:(k + 1) * r] -= LR * grad[k] / case["n_dirs"] * _factor(seeds[k], 2 * i, case["m"], r, True)
            out.append(P)
        return {"cand_loss": loss, "proj_grad": grad, "P": out}
    nq, nkv = case["heads"] * 128, case["kv"] * 128
    q, k, v = x["qkv"][:, :nq], x["qkv"][:, nq:nq + nkv], x["qkv"][:, nq + nkv:]
    if kind == "attn":
        return {"O": _exact_attention(pk, q, k, v, case["heads"], case["kv"])}
    h = x["X"].double() + x["res"].double()
    hb = h.to(torch.bfloat16).double()   # the stored sum is what is normalised
    return {"hsum": h, "y": _exact_norm(hb, x["gamma"], x["beta"], case["norm"]),
            "qkv": torch.cat([_exact_rope(pk, q, x["gq"]), _exact_rope(pk, k, x["gk"]), v.double()], 1)}
