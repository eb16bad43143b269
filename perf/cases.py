"""The calls whose speed is measured: what a program that generates with the
speculative-decoding library makes it do, through its public entry points.

Sizes are those of the configured pairs (``workloads/configs.py``): a tiny fp32
decoder, a small bf16 one, an 8B-shaped target and its 1B-shaped drafter.  Six
kinds of case:

* ``draw``         the drafter's draw from its own logits (``spec_sample_draft``)
* ``decide``       acceptance scan, residual resample and bonus draw on caller
                   logits (``spec_sample_verify``; ``_noalloc`` with device inputs)
* ``gemm``         one decoder projection (``spec_op_gemm``)
* ``attn``         paged causal attention of one layer (``spec_op_attention``)
* ``verify``       a session's verify round: target forward over every
                   sequence's k + 1 rows and the decision, commit, rollback
                   (``forward``: the batched target forward alone)
* ``first_token``  a prompt's prefill and the forward of its pending token

``exact`` is the same arithmetic in float64 torch, written out here.
"""

import math

import numpy as np
import torch

from paper_2607_20507_amd import binding as B
from paper_2607_20507_amd.session import DeviceModel, SpecSession
from workloads import configs as C

MODELS = {"tiny": C.TINY_TARGET, "small": C.SMALL_TARGET, "1b": C.L1B_DRAFT, "8b": C.L8B_TARGET}
DEV = "cuda"


def listed():
    return [
        # the draw of one draft step of the small pair's 8 sequences: the smallest call, all latency
        {"name": "draw_small", "kind": "draw", "n": 8, "vocab": 32000, "temperature": 0.7},
        # the decision pass of a large batch on its own: 256 sequences x 8 rows, the vocab-stress workload
        {"name": "decide_stress", "kind": "decide", "batch": 256, "k": 7, "vocab": 128256, "noalloc": False, "greedy": 0.0},
        # the largest weight of a single sequence's verify (6 rows): gate / up of the 8B-shaped target
        {"name": "gemm_single_gate_up", "kind": "gemm", "model": "8b", "proj": "gate_up", "rows": 6},
        # the same projection in the 64-sequence verify (k drawn from 3, 5, 7: 364 rows)
        {"name": "gemm_serving_gate_up", "kind": "gemm", "model": "8b", "proj": "gate_up", "rows": 364},
        # and in a long prompt's prefill chunk
        {"name": "gemm_prefill_gate_up", "kind": "gemm", "model": "8b", "proj": "gate_up", "rows": 8192},
        # one layer's attention of the 64-sequence verify over contexts of 512 to 4096 tokens
        {"name": "attn_serving", "kind": "attn", "model": "8b", "batch": 64, "rows": 0, "context": 0},
        # one layer's attention of an 8192-token prompt's prefill
        {"name": "attn_prefill", "kind": "attn", "model": "8b", "batch": 1, "rows": 8192, "context": 8192},
        # the tiny fp32 pair's verify round: fp32 kernels, all launch latency
        {"name": "verify_tiny_fp32", "kind": "verify", "model": "tiny", "layers": 2, "batch": 1, "context": 128, "k": 4, "forward": False},
        # the small pair as configured: 12 layers, 8 sequences of 256 to 512 tokens, k = 5
        {"name": "verify_small", "kind": "verify", "model": "small", "layers": 12, "batch": 8, "context": 0, "k": 5, "forward": False},
        # the headline call: one sequence's verify round on the 8B-shaped target, context 2048, k = 5 (8 of the
        # layers: over all 32 the roundings of two correct bf16 passes drift further apart than a tolerance is worth)
        {"name": "verify_single_8b", "kind": "verify", "model": "8b", "layers": 8, "batch": 1, "context": 2048, "k": 5, "forward": False},
        # the parallel-serving verify's target forward: 64 sequences, contexts of 512 to 4096 (4 of the layers)
        {"name": "forward_serving_8b", "kind": "verify", "model": "8b", "layers": 4, "batch": 64, "context": 0, "k": 0, "forward": True},
        # a 4096-token prompt up to its first token (4 of the layers)
        {"name": "first_token_8b", "kind": "first_token", "model": "8b", "layers": 4, "prompt": 4096},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["draw", "decide", "gemm", "gemm", "attn", "attn", "verify", "first_token"])
    if kind == "draw":
        return {"kind": "draw", "n": _log(rng, 1, 64), "vocab": rng.choice([32000, 128256, _log(rng, 1000, 128256)]),
                "temperature": rng.choice([0.0, 0.7, 0.8, 1.0])}
    if kind == "decide":
        return {"kind": "decide", "batch": _log(rng, 1, 256), "k": rng.randint(1, 7),
                "vocab": rng.choice([32000, 128256, _log(rng, 1000, 128256)]), "noalloc": rng.random() < 0.5,
                "greedy": rng.choice([0.0, 0.0, 0.25, 1.0])}
    if kind == "gemm":
        model = rng.choice(["tiny", "small", "1b", "1b", "8b", "8b"])
        proj = rng.choice(["qkv", "o", "gate_up", "down", "lm_head"])
        most = {"tiny": 512, "small": 4096, "1b": 8192, "8b": 6000}[model] if proj != "lm_head" else 512
        return {"kind": "gemm", "model": model, "proj": proj, "rows": _log(rng, 1, most)}
    if kind == "attn":
        model = rng.choice(["tiny", "small", "1b", "8b", "8b"])
        if rng.random() < 0.4 and model != "tiny":  # prefill
            rows = _log(rng, 64, 6000)
            return {"kind": "attn", "model": model, "batch": 1, "rows": rows, "context": rows + rng.choice([0, 0, rng.randint(0, 1000)])}
        return {"kind": "attn", "model": model, "batch": _log(rng, 1, 8 if model == "tiny" else 64), "rows": rng.randint(1, 8),
                "context": _log(rng, 64, 512 if model == "tiny" else 4096)}
    if kind == "verify":
        model = rng.choice(["tiny", "small", "1b", "8b"])
        return {"kind": "verify", "model": model, "layers": {"tiny": 2, "small": 12, "1b": 16, "8b": 4}[model],
                "batch": _log(rng, 1, 4 if model == "tiny" else 24), "context": _log(rng, 64, 300 if model == "tiny" else 1500),
                "k": rng.randint(1, 7), "forward": rng.random() < 0.5}
    model = rng.choice(["small", "1b", "8b"])
    return {"kind": "first_token", "model": model, "layers": {"small": 12, "1b": 16, "8b": 4}[model], "prompt": _log(rng, 16, 3500)}


# ---------------------------------------------------------------------------
# inputs

def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1_000_033 + tag)
    return g


def _dtype(sh):
    return torch.float32 if sh.dtype == "f32" else torch.bfloat16


def _code(sh):
    return B.SPEC_F32 if sh.dtype == "f32" else B.SPEC_BF16


def _lens(case, seed):
    """Context length (prompt tokens) and draft count of each sequence."""
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 11])
    n = case["batch"]
    if case["context"]:
        ctx = [case["context"]] * n
        if n > 1:  # a batch's contexts differ
            ctx = [int(x) for x in rng.integers(max(2, case["context"] // 2), case["context"] + 1, n)]
    elif case["model"] == "small":
        ctx = [int(x) for x in rng.integers(256, 513, n)]
    else:  # log-uniform over the octave midpoints, so that every seed has about the same total
        ctx = [int(512 * 8 ** ((i + rng.uniform()) / n)) for i in range(n)]
    k = case.get("k", 0) or case.get("rows", 0)
    if case["kind"] == "verify":
        ks = [k] * n if k else [(3, 5, 7)[i % 3] for i in range(n)]
    else:
        ks = [k - 1] * n if k else [(3, 5, 7)[i % 3] for i in range(n)]
    return ctx, ks


def _gemm_shape(case):
    """(N, K, epilogue) of a projection."""
    sh = MODELS[case["model"]]
    return {"qkv": (sh.qkv_rows, sh.d_model, B.SPEC_EPI_STORE_F32),
            "o": (sh.d_model, sh.q_dim, B.SPEC_EPI_ADD_F32),
            "gate_up": (sh.ffn_dim, sh.d_model, B.SPEC_EPI_SWIGLU),
            "down": (sh.d_model, sh.ffn_dim, B.SPEC_EPI_ADD_F32),
            "lm_head": (sh.vocab, sh.d_model, B.SPEC_EPI_STORE_F32)}[case["proj"]]


def _gemm_inputs(case, seed):
    """X (normed rows; the products of gate and up for the down projection), W row-major, residual rows."""
    sh = MODELS[case["model"]]
    N, K, epi = _gemm_shape(case)
    g = _gen(seed, 1)
    Nw = 2 * N if epi == B.SPEC_EPI_SWIGLU else N
    x = torch.randn(case["rows"], K, generator=g, device=DEV)
    if case["proj"] in ("down", "o"):
        x *= 0.5
    w = torch.empty(Nw, K, dtype=_dtype(sh), device=DEV)
    step = max(1, (1 << 26) // K)
    for s in range(0, Nw, step):
        e = min(Nw, s + step)
        w[s:e] = (torch.randn(e - s, K, generator=g, device=DEV) * sh.init_std).to(w.dtype)
    h = torch.randn(case["rows"], N, generator=g, device=DEV) if epi == B.SPEC_EPI_ADD_F32 else None
    return x.to(w.dtype), w, h


def _attn_shape(case, seed):
    """Query rows and first position of each sequence, pages per sequence."""
    if case["rows"] >= 64 and case["batch"] == 1:
        rows, pos0 = [case["rows"]], [case["context"] - case["rows"]]
    else:
        ctx, ks = _lens(case, seed)
        rows = [k + 1 for k in ks]
        pos0 = [max(0, c - 1) for c in ctx]
    return rows, pos0, max((p + r + 15) // 16 for p, r in zip(pos0, rows))


def _attn_inputs(case, seed):
    sh = MODELS[case["model"]]
    rows, pos0, mp = _attn_shape(case, seed)
    need = [(p + r + 15) // 16 for p, r in zip(pos0, rows)]
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 12])
    perm = rng.permutation(sum(need)).astype(np.int32)
    pt = np.zeros((len(rows), mp), dtype=np.int32)
    o = 0
    for i, n in enumerate(need):
        pt[i, :n] = perm[o:o + n]
        o += n
    g = _gen(seed, 2)
    blk = (sum(need), sh.n_kv_heads, 16, sh.head_dim)
    q = torch.randn(sum(rows), sh.n_heads, sh.head_dim, generator=g, device=DEV).to(_dtype(sh))
    kp = torch.randn(blk, generator=g, device=DEV).to(_dtype(sh))
    vp = torch.randn(blk, generator=g, device=DEV).to(_dtype(sh))
    return rows, pos0, pt, q, kp, vp


def _prompts(case, seed, lens):
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 13])
    V = MODELS[case["model"]].vocab
    return [rng.integers(0, V, n, dtype=np.int32) for n in lens]


def _drafts(case, seed, ks):
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 14])
    V = MODELS[case["model"]].vocab
    return [rng.integers(0, V, k, dtype=np.int32) for k in ks]


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case, s.seed = case, int(seed)
    kind = case["kind"]
    if kind == "draw":
        n, V = case["n"], case["vocab"]
        s.logits = torch.randn(n, V, generator=_gen(seed, 3), device=DEV)
        s.temps = np.full(n, case["temperature"], dtype=np.float32)
        s.ids = np.arange(1, n + 1, dtype=np.int64)
        s.pos = np.arange(300, 300 + n, dtype=np.int32)
        s.tokens = torch.zeros(n, dtype=torch.int32, device=DEV)
        s.ws = torch.empty(B.spec_sample_workspace_bytes(n, max(n, 2 * n), V) + (1 << 20), dtype=torch.uint8, device=DEV)
    elif kind == "decide":
        _prepare_decide(s, case, seed)
    elif kind == "gemm":
        sh = MODELS[case["model"]]
        s.N, s.K, s.epi = _gemm_shape(case)
        s.dt = _code(sh)
        s.x, s.w, s.h = _gemm_inputs(case, seed)
        if sh.dtype == "bf16":
            if s.epi == B.SPEC_EPI_SWIGLU:
                B.spec_pack_weight(s.w[:s.N], s.N, s.K)
                B.spec_pack_weight(s.w[s.N:], s.N, s.K)
            else:
                B.spec_pack_weight(s.w, s.N, s.K)
        R = case["rows"]
        s.y = torch.zeros(R, s.N, dtype=s.w.dtype if s.epi == B.SPEC_EPI_SWIGLU else torch.float32, device=DEV)
        s.ws = torch.empty(B.spec_op_gemm_workspace_bytes(R, s.w.shape[0]), dtype=torch.uint8, device=DEV)
    elif kind == "attn":
        sh = MODELS[case["model"]]
        s.rows, s.pos0, s.pt, s.q, s.kp, s.vp = _attn_inputs(case, seed)
        s.shape = (_code(sh), sh.n_heads, sh.n_kv_heads, sh.head_dim)
        s.out = torch.zeros(s.q.shape[0], sh.q_dim, dtype=s.q.dtype, device=DEV)
        s.ws = torch.empty(B.spec_op_attention_workspace_bytes(len(s.rows), s.q.shape[0], s.pt.shape[1], sh.n_kv_heads,
                                                               sh.head_dim) + 8192, dtype=torch.uint8, device=DEV)
    elif kind == "verify":
        ctx, ks = _lens(case, seed)
        kmax = max(ks)
        s.model = DeviceModel(MODELS[case["model"]], device=DEV, seed=s.seed, n_layers=case["layers"])
        s.sess = SpecSession(s.model, None, max_seqs=len(ctx), k_max=kmax, max_pages_per_seq=(max(ctx) + kmax + 16) // 16 + 1,
                             num_pages_target=sum((c + kmax + 16) // 16 + 1 for c in ctx), max_rows=8192)
        s.ids = list(range(1, len(ctx) + 1))
        s.len = [c - 1 for c in ctx]
        s.temps = [0.8] * len(ctx)
        s.sess.prefill(s.ids, _prompts(case, seed, ctx))
        s.drafts = _drafts(case, seed, ks)
        s.q = torch.randn(kmax, s.model.shape.vocab, generator=_gen(seed, 4), device=DEV)
        for i, t in zip(s.ids, s.drafts):
            s.sess.set_drafts(i, t, s.q)
    else:
        P = case["prompt"]
        s.model = DeviceModel(MODELS[case["model"]], device=DEV, seed=s.seed, n_layers=case["layers"])
        s.sess = SpecSession(s.model, None, max_seqs=1, k_max=1, max_pages_per_seq=(P + 32) // 16, max_rows=8192)
        s.prompt = _prompts(case, seed, [P])
    return s


def _prepare_decide(s, case, seed):
    b, k, V = case["batch"], case["k"], case["vocab"]
    g = _gen(seed, 5)
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 15])
    if case["noalloc"]:
        ks = rng.integers(max(1, k - 2), k + 1, b).astype(np.int32)
        ks[0] = k
    else:
        ks = np.full(b, k, dtype=np.int32)
    temps = np.array([0.0 if rng.uniform() < case["greedy"] else (0.3, 1.0, 1.5)[i % 3] for i in range(b)], dtype=np.float32)
    s.ks, s.temps = ks, temps
    s.ids = np.arange(1, b + 1, dtype=np.int64) * 7
    s.base = rng.integers(512, 4096, b).astype(np.int32)
    s.p = torch.randn(int(ks.sum()) + b, V, generator=g, device=DEV) * 3.0
    s.q = torch.empty(int(ks.sum()), V, device=DEV)
    s.tok = torch.empty(int(ks.sum()), dtype=torch.int32, device=DEV)
    pr = qr = 0
    for i in range(b):  # q = p + N(0, 1), drafts drawn from softmax(q / T)
        n = int(ks[i])
        z = s.p[pr:pr + n] + torch.randn(n, V, generator=g, device=DEV)
        s.q[qr:qr + n] = z
        t = float(temps[i])
        if t > 0:
            z = z / t - torch.empty_like(z).exponential_(generator=g).log()
        s.tok[qr:qr + n] = z.argmax(dim=1).int()
        pr += n + 1
        qr += n
    s.nacc = torch.zeros(b, dtype=torch.int32, device=DEV)
    s.otok = torch.zeros(b, k + 1, dtype=torch.int32, device=DEV)
    s.ws = torch.empty(B.spec_sample_workspace_bytes(b, s.p.shape[0] + s.q.shape[0], V) + (1 << 20), dtype=torch.uint8, device=DEV)
    if case["noalloc"]:
        s.dk, s.dt = torch.from_numpy(ks).to(DEV), torch.from_numpy(temps).to(DEV)
        s.dids, s.dbase = torch.from_numpy(s.ids).to(DEV), torch.from_numpy(s.base).to(DEV)


# ---------------------------------------------------------------------------
# one pass

def _logits(sess):
    """The last forward's logits, in the session's own buffer."""
    ptr, rows = B.spec_last_logits(sess.ctx)
    V = sess.target.shape.vocab
    off = ptr - sess.ws_view.data_ptr()
    return sess.ws_view[off:off + rows * V * 4].view(torch.float32).view(rows, V)


def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "draw":
        B.spec_sample_draft(s.logits, case["vocab"], s.temps, s.ids, s.pos, s.seed, s.tokens, s.ws)
        return s.tokens
    if kind == "decide":
        if case["noalloc"]:
            B.spec_sample_verify_noalloc(case["k"], s.dk, s.dt, s.dids, s.dbase, s.p, s.q, s.tok, case["vocab"], s.seed, s.nacc, s.otok)
        else:
            B.spec_sample_verify(s.ks, s.temps, s.ids, s.base, s.p, s.q, s.tok, case["vocab"], s.seed, s.nacc, s.otok, s.ws)
        return s.nacc, s.otok
    if kind == "gemm":
        if s.h is not None:  # the residual rows the projection adds to
            s.y.copy_(s.h)
        B.spec_op_gemm(s.dt, case["rows"], s.N, s.K, s.x, s.w, s.y, s.epi, s.ws)
        return s.y
    if kind == "attn":
        dt, hq, hkv, hd = s.shape
        B.spec_op_attention(dt, s.rows, s.pos0, s.pt, hq, hkv, hd, s.q, s.kp, s.vp, s.out, s.ws)
        return s.out
    if kind == "verify":
        if case["forward"]:
            s.sess.target_forward(s.ids)
            return _logits(s.sess)
        # a round whose tokens the caller drops again, so that every pass is the same round
        na, _ = s.sess.verify(s.ids, s.temps, s.seed)
        s.sess.commit(s.ids, na)
        for i, n, t in zip(s.ids, s.len, s.drafts):
            s.sess.rollback(i, n)
            s.sess.set_drafts(i, t, s.q)
        return _logits(s.sess)
    s.sess.prefill([1], s.prompt)
    s.sess.target_forward([1])
    s.sess.release(1)
    return _logits(s.sess)


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct passes may be apart

def _layer_weights(sh):
    d = sh.d_model
    return sh.qkv_rows * d + d * sh.q_dim + 3 * sh.ffn_dim * d


def work(case):
    kind = case["kind"]
    if kind == "draw":
        return {"bytes": 4.0 * case["n"] * case["vocab"] + 4 * case["n"], "flops": 4.0 * case["n"] * case["vocab"]}
    if kind == "decide":
        rows = case["batch"] * (2 * case["k"] + 1)
        return {"bytes": 4.0 * rows * case["vocab"], "flops": 4.0 * rows * case["vocab"]}
    sh = MODELS[case["model"]]
    esz = sh.bytes_per_elem()
    if kind == "gemm":
        N, K, epi = _gemm_shape(case)
        Nw, R = (2 * N if epi == B.SPEC_EPI_SWIGLU else N), case["rows"]
        out = {B.SPEC_EPI_STORE_F32: 4, B.SPEC_EPI_ADD_F32: 8, B.SPEC_EPI_SWIGLU: esz}[epi]
        return {"bytes": float(esz) * (Nw * K + R * K) + float(out) * R * N, "flops": 2.0 * R * Nw * K}
    if kind == "attn":
        rows, pos0, _ = _attn_shape(case, 1)
        keys = sum(p + r for p, r in zip(pos0, rows))
        qk = sum(r * p + r * (r + 1) / 2 for p, r in zip(pos0, rows))
        return {"bytes": esz * (2.0 * keys * sh.kv_dim + 2.0 * sum(rows) * sh.q_dim), "flops": 4.0 * qk * sh.q_dim}
    L = case["layers"]
    if kind == "verify":
        ctx, ks = _lens(case, 1)
        R = sum(ks) + len(ks)
        keys = sum(c + k for c, k in zip(ctx, ks))
        qk = sum((k + 1) * c for c, k in zip(ctx, ks))
        wb = float(esz) * (L * _layer_weights(sh) + sh.vocab * sh.d_model)
        logits = 4.0 * R * sh.vocab
        if not case["forward"]:  # the decision reads the target rows written just before it and the draft rows
            logits += 4.0 * (R + sum(ks)) * sh.vocab
        return {"bytes": wb + logits + 2.0 * esz * L * keys * sh.kv_dim + float(esz) * R * sh.d_model,
                "flops": 2.0 * R * (L * _layer_weights(sh) + sh.vocab * sh.d_model) + 4.0 * L * qk * sh.q_dim}
    P = case["prompt"]
    return {"bytes": float(esz) * (L * _layer_weights(sh) + sh.vocab * sh.d_model) + 2.0 * esz * L * P * sh.kv_dim
            + 4.0 * sh.vocab + float(esz) * P * sh.d_model,
            "flops": 2.0 * P * L * _layer_weights(sh) + 2.0 * sh.vocab * sh.d_model + 2.0 * L * P * P * sh.q_dim}


def tolerance(case):
    kind = case["kind"]
    if kind in ("draw", "decide"):
        # tokens and counts: a draw flips only where two scores agree to the last bits of fp32
        return {"rel": 0.0, "differ": 0.01}
    f32 = MODELS[case["model"]].dtype == "f32"
    if kind == "gemm":
        if f32 or _gemm_shape(case)[2] != B.SPEC_EPI_SWIGLU:
            return {"rel": 4e-6}  # fp32 sums of up to 14336 products: 3e-7 from float64
        return {"rel": 4e-3}      # bf16 results: half a unit in the last place each, 1.7e-3 in the 2-norm
    if kind == "attn":
        return {"rel": 4e-6 if f32 else 8e-3}  # bf16: probabilities and results rounded to 8 bits, 2.1e-3 from float64
    # whole forwards: a layer's roundings travel through the layers after it (from float64: fp32 8e-7, the
    # small pair's 12 layers 7e-3, 4 layers of the 8B-shaped target 1.5e-2)
    return {"rel": 4e-6 if f32 else 1.5e-2 if case["model"] == "small" else 2.5e-2}


# ---------------------------------------------------------------------------
# float64

def _pages_to_rows(blk, sh):
    """(K, V) pages [n, Hkv, 16, hd] in the library's documented orders -> index maps [16, hd] into a block."""
    hd = sh.head_dim
    k = torch.arange(16, device=DEV)[:, None]
    d = torch.arange(hd, device=DEV)[None, :]
    if sh.dtype == "f32":
        return k * hd + d, d * 16 + k
    c = d // 8
    ki = 8 * ((((c // 4) * 2 + (k // 4) % 2) * 4 + c % 4) * 8 + k % 4 + 4 * (k // 8)) + d % 8
    vi = 8 * (((d // 16) * 2 + k // 8) * 16 + d % 16) + k % 8
    return ki, vi


def _attend(q, k, v, pos0, limit=1 << 27):
    """Causal attention in float64: q [R, Hq, hd] at positions pos0.., k and v [T, Hkv, hd]."""
    R, hq, hd = q.shape
    T, hkv, _ = k.shape
    G = hq // hkv
    out = torch.empty_like(q)
    step = max(1, limit // max(1, T * G))
    for h in range(hkv):
        kh, vh = k[:, h].contiguous(), v[:, h].contiguous()
        for a in range(0, R, step):
            e = min(R, a + step)
            t = pos0 + e  # keys any of these rows sees
            qq = q[a:e, h * G:(h + 1) * G].reshape(-1, hd)
            z = qq @ kh[:t].t().contiguous() / math.sqrt(hd)
            lim = (pos0 + torch.arange(a, e, device=q.device)).repeat_interleave(G)
            z.masked_fill_(torch.arange(t, device=q.device)[None, :] > lim[:, None], -math.inf)
            out[a:e, h * G:(h + 1) * G] = (torch.softmax(z, dim=1) @ vh[:t]).view(e - a, G, hd)
    return out


def _weights(sh, seed, tag, rows, cols):
    """A weight as DeviceModel draws it from its seed."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1_000_003 + tag)
    out = torch.empty(rows, cols, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // cols)
    for s in range(0, rows, step):
        e = min(rows, s + step)
        out[s:e] = (torch.randn(e - s, cols, generator=g, device=DEV) * sh.init_std).to(_dtype(sh)).double()
    return out


def _forward64(sh, seed, L, seqs, last):
    """float64 logits of the last last[i] positions of each token list."""
    d, hd, f = sh.d_model, sh.head_dim, sh.ffn_dim
    E = _weights(sh, seed, 7_000_001, sh.vocab, d)
    hs = [E[torch.from_numpy(np.asarray(t, dtype=np.int64)).to(DEV)] for t in seqs]
    del E

    def norm(x):
        return x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + sh.rms_eps)

    freq = sh.rope_theta ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)

    def rope(x):
        a = torch.arange(x.shape[0], device=DEV, dtype=torch.float64)[:, None] * freq
        c, s = a.cos()[:, None], a.sin()[:, None]
        u, w = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([u * c - w * s, w * c + u * s], dim=-1)

    for l in range(L):
        wqkv = _weights(sh, seed, 10 * l + 1, sh.qkv_rows, d).t().contiguous()
        wo = _weights(sh, seed, 10 * l + 2, d, sh.q_dim).t().contiguous()
        wgu = _weights(sh, seed, 10 * l + 3, 2 * f, d).t().contiguous()
        wd = _weights(sh, seed, 10 * l + 4, d, f).t().contiguous()
        for i, h in enumerate(hs):
            x = (norm(h) @ wqkv).view(h.shape[0], -1, hd)
            q, k, v = x[:, :sh.n_heads], x[:, sh.n_heads:sh.n_heads + sh.n_kv_heads], x[:, sh.n_heads + sh.n_kv_heads:]
            h = h + _attend(rope(q).contiguous(), rope(k), v, 0).reshape(h.shape[0], -1) @ wo
            gu = norm(h) @ wgu
            hs[i] = h + (torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]) @ wd
    rows = torch.cat([norm(h[-n:]) for h, n in zip(hs, last)])
    lm = _weights(sh, seed, 7_000_002, sh.vocab, d)
    return rows @ lm.t().contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("draw", "decide"):
        return None  # whole values
    sh = MODELS[case["model"]]
    if kind == "gemm":
        N, K, epi = _gemm_shape(case)
        x, w, h = _gemm_inputs(case, seed)
        x = x.double()
        y = torch.empty(x.shape[0], w.shape[0], dtype=torch.float64, device=DEV)
        for s in range(0, w.shape[0], 16384):
            y[:, s:s + 16384] = x @ w[s:s + 16384].double().t().contiguous()
        if epi == B.SPEC_EPI_SWIGLU:
            return torch.nn.functional.silu(y[:, :N]) * y[:, N:]
        return y + h.double() if h is not None else y
    if kind == "attn":
        rows, pos0, pt, q, kp, vp = _attn_inputs(case, seed)
        ki, vi = _pages_to_rows(kp, sh)
        out = torch.empty(q.shape[0], sh.q_dim, dtype=torch.float64, device=DEV)
        r0 = 0
        for i, (r, p) in enumerate(zip(rows, pos0)):
            t = p + r
            pages = torch.from_numpy(pt[i, :(t + 15) // 16].astype(np.int64)).to(DEV)

            def rows_of(pool, idx):
                b = pool[pages].view(len(pages), sh.n_kv_heads, -1)[:, :, idx.reshape(-1)].double()
                return b.view(len(pages), sh.n_kv_heads, 16, sh.head_dim).transpose(1, 2).reshape(-1, sh.n_kv_heads, sh.head_dim)[:t]

            out[r0:r0 + r] = _attend(q[r0:r0 + r].double(), rows_of(kp, ki), rows_of(vp, vi), p).reshape(r, -1)
            r0 += r
        return out
    if kind == "verify":
        ctx, ks = _lens(case, seed)
        seqs = [np.concatenate([p, t]) for p, t in zip(_prompts(case, seed, ctx), _drafts(case, seed, ks))]
        return _forward64(sh, seed, case["layers"], seqs, [k + 1 for k in ks])
    return _forward64(sh, seed, case["layers"], _prompts(case, seed, [case["prompt"]]), [1])
