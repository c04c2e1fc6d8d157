"""The work a program has this library do, as cases that can be timed and checked.

A case is a dict of plain values; `prepare` makes what a program holds before the call (weights, a loaded
model, a prefilled session, a KV pool), `run` is one pass through the public entry points.  Two sorts:

* single layers and blocks: a decode projection (`projection`), the gate / up sweep with its SwiGLU
  (`gate_up`), a head evaluation (`head`), the prompt-pass projection (`gemm`), attention of the decode path
  (`attention`) and of the prompt (`prompt_attention`);
* calls on a model: prompts (`prefill`), decoding with the paper's rounds (`decode`), one round of sampling-mode
  verification (`sampled`), several sequences together (`batch`), and the whole of a small fp32 model
  (`generate`).  The models have the layer shapes of the benchmark configurations with fewer layers, so that
  weights are made quickly; everything a layer does is there.

Weights are N(0, 0.02) (output projections less, as in sb_inputs.make_weights), prompts uniform ids.
"""
from dataclasses import replace
import math

import numpy as np
import torch

import paper_2604_12247_amd as sb
import sb_inputs as si

DEV = "cuda"
PAGE = sb.SB_KV_BLOCK
PROJ = {"packed": sb.PROJ_MFMA_PACKED, "rows": sb.PROJ_MFMA, "valu": sb.PROJ_VALU}
SHAPES = {"7b": si.CONFIGS["C2"].shape, "13b": si.CONFIGS["C4"].shape, "8b": si.CONFIGS["C5"].shape,
          "tiny": si.CONFIGS["C1"].shape}


def listed():
    return [
        # a small fp32 model, whole: 32 prompt tokens and 64 new ones with forced exits (latency and launches count)
        dict(name="generate_tiny_fp32", kind="generate", shape="tiny", layers=4, heads=2, prompt=32, new=64, w=4),
        # the headline: rounds of six drafts and their verification at the 7B shape behind a 512-token prompt
        dict(name="decode_7b_rounds", kind="decode", shape="7b", layers=6, heads=3, prompt=512, rounds=8, w=6, mode="forced"),
        # sampling-mode verification (temperature, top-p) of a round at the 8B grouped-query shape, V = 128256
        dict(name="sampled_8b_round", kind="sampled", shape="8b", layers=2, heads=1, prompt=700, w=4, temp=0.3, top_p=0.9),
        # four sequences decoded together at the 13B shape, contexts of different lengths
        dict(name="batch4_13b", kind="batch", shape="13b", layers=3, heads=0, prompt=300, rounds=12, w=1, batch=4),
        # prompts: a chat turn, the benchmark's 512 tokens, a ragged long one
        dict(name="prefill_13b_45", kind="prefill", shape="13b", layers=4, prompt=45),
        dict(name="prefill_7b_512", kind="prefill", shape="7b", layers=4, prompt=512),
        dict(name="prefill_8b_1999", kind="prefill", shape="8b", layers=4, prompt=1999),
        # one exit head of a draft step at the 7B shape
        dict(name="head_7b", kind="head", N=32000, K=4096, M=1, kernel="packed", T=1.4),
        # gate / up of a six-row verification pass at the 13B shape
        dict(name="gate_up_13b_m6", kind="gate_up", N=13824, K=5120, M=6, kernel="packed"),
        # QKV of a greedy token at the grouped-query shape: the smallest projection of the three models
        dict(name="qkv_8b_m1", kind="projection", N=6144, K=4096, M=1, kernel="packed", fp32=False),
        # attention of a verification pass over a long context, and of a 4096-token prompt's second half
        dict(name="attention_7b_4200", kind="attention", q=32, kv=32, hd=128, pos=4200, M=6, fp32=False),
        dict(name="prompt_attention_7b_4096", kind="prompt_attention", q=32, kv=32, hd=128, pos=2048, M=2048),
    ]


def draw(rng):
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["projection", "gate_up", "head", "gemm", "attention", "attention", "prompt_attention", "prefill",
                       "prefill", "decode", "sampled", "batch", "generate"])
    big = rng.choice(["7b", "13b", "8b"])
    if kind in ("projection", "gate_up", "head"):
        kernel = rng.choice(["packed", "packed", "packed", "rows", "valu"])
        c = dict(kind=kind, N=16 * logu(32, 1000), K=128 * logu(4, 110), M=rng.randint(1, 8), kernel=kernel)
        if kind == "projection":
            c["fp32"] = kernel == "valu" and rng.random() < 0.5
        if kind == "head":
            c.update(N=16 * logu(100, 8016), K=128 * rng.randint(8, 40), T=round(rng.uniform(0.7, 2.0), 2))
        return c
    if kind == "gemm":
        return dict(kind=kind, N=16 * logu(64, 2000), K=128 * logu(8, 110), M=rng.randint(9, 128))
    if kind in ("attention", "prompt_attention"):
        hd, kv = rng.choice([64, 128]), rng.choice([4, 8, 32, 40])
        q = kv if kv > 8 else kv * rng.choice([2, 4, 8])
        if kind == "attention":
            return dict(kind=kind, q=q, kv=kv, hd=hd, pos=logu(5, 9000), M=rng.randint(1, 8), fp32=rng.random() < 0.15)
        return dict(kind=kind, q=q, kv=kv, hd=hd, pos=rng.choice([0, 0, logu(1, 2000)]), M=logu(9, 2048))
    if kind == "prefill":
        return dict(kind=kind, shape=big, layers=rng.randint(2, 4), prompt=logu(9, 1300))
    if kind == "decode":
        return dict(kind=kind, shape=big, layers=rng.randint(4, 5), heads=2, prompt=logu(20, 1500), rounds=rng.randint(4, 7),
                    w=rng.randint(2, 6), mode=rng.choice(["greedy", "forced", "computed"]))
    if kind == "sampled":
        return dict(kind=kind, shape=big, layers=2, heads=1, prompt=logu(20, 1000), w=rng.randint(1, 6),
                    temp=rng.choice([0.25, 0.3]), top_p=rng.choice([0.9, 0.9, 1.0]))
    if kind == "batch":
        b = rng.choice([2, 3, 4, 8])
        return dict(kind=kind, shape=big, layers=3, heads=1, prompt=logu(20, 600), rounds=rng.randint(5, 10),
                    w=rng.randint(1, 8 // b), batch=b)
    return dict(kind="generate", shape="tiny", layers=rng.randint(2, 6), heads=1, prompt=rng.randint(5, 90),
                new=rng.randint(16, 64), w=rng.randint(1, 6))


# ---------------------------------------------------------------- seeded inputs
def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + what * 7919 + 12345) % (1 << 62))
    return g


def _normal(seed, what, shape, std=1.0, fp32=True):
    x = torch.randn(shape, generator=_gen(seed, what), device=DEV, dtype=torch.float32)
    x *= std
    return x if fp32 else x.to(torch.bfloat16)


def _ids(seed, what, n, vocab):
    return torch.randint(0, vocab, (n,), generator=_gen(seed, what), device=DEV).cpu().numpy().astype(np.int32)


def _shape(case):
    return replace(SHAPES[case["shape"]], n_layers=case["layers"], n_exit_heads=case.get("heads", 0))


def _device_weights(case, s, seed):
    """{name: tensor on the GPU}: matrices in the model's weight type, norm gains jittered around 1."""
    fp32 = s.weight_dtype == si.configs.FP32
    w = {}
    for i, (name, shp, std) in enumerate(si.tensor_specs(s)):
        w[name] = _normal(seed, 100 + i, shp, std, fp32)
    norms = ["final_norm"] + [f"{n}.{l}" for l in range(s.n_layers) for n in ("attn_norm", "ffn_norm")]
    for i, name in enumerate(norms + [f"exit_norm.{l}" for l in range(s.n_exit_heads)]):
        w[name] = 1.0 + 0.1 * _normal(seed, 5000 + i, (s.d_model,))
    if case.get("mode") == "computed":
        # exits decided by the confidences need heads that agree with the model: deeper layers refine less, the
        # exit heads are the final head, made peaked
        for l in range(s.n_layers):
            w[f"w_o.{l}"] *= 0.5 ** l
            w[f"w_down.{l}"] *= 0.5 ** l
        for l in range(s.n_exit_heads):
            w[f"exit_head.{l}"], w[f"exit_norm.{l}"] = w["lm_head"], w["final_norm"] * 4.0
    return w


def _host(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return (h.view(torch.int16) if h.dtype == torch.bfloat16 else h).numpy()


def _capacity(case):
    n = case["prompt"] + case.get("batch", 1) * 3 + case.get("new", case.get("rounds", 0)) + 2 * case.get("w", 0) + 24
    return (n + PAGE - 1) // PAGE * PAGE


def _model(case, seed):
    s = _shape(case)
    w = _device_weights(case, s, seed)
    host = {k: _host(v) for k, v in w.items()}
    del w
    return s, sb.Model(s, host, _capacity(case))


def _temps(n):
    return [2.0 - l / max(n - 1, 1) for l in range(n)]


def _exits(case, seed, n):
    """Forced exit layers, one a draft step."""
    return np.random.default_rng(seed + 17).integers(1, case["heads"] + 1, n).astype(np.int32)


def _script(case, seed, b=0):
    """The tokens that decoding is made to follow, whatever the model's own choices: fed and drafted ids.  (A greedy
    choice between two near-equal logits of random weights may fall either way; what follows it would differ.)"""
    return _ids(seed, 50 + b, case["rounds"] + case["w"], SHAPES[case["shape"]].vocab)


def _prompt(case, seed, b=0):
    return _ids(seed, 10 + b, case["prompt"] + 3 * b, SHAPES[case["shape"]].vocab)


def _params(case, seed, script):
    """Rounds that start at any token of the script and draft the ones after it."""
    w, d = case["w"], case["heads"]
    if case.get("mode") == "greedy" or (case["kind"] == "batch" and w == 1):
        return sb.Params(0, 1, [], 2.0)
    if case.get("mode") == "computed":
        return sb.Params(d, w, _temps(d), 0.4)
    fd = np.concatenate([script[r + 1:r + 1 + w] for r in range(case["rounds"])])
    return sb.Params(d, w, _temps(d), 2.0, forced_exit=_exits(case, seed, len(fd)), forced_draft=fd)


def _attention_inputs(case, seed):
    hd, kv, q, M, pos = case["hd"], case["kv"], case["q"], case["M"], case["pos"]
    fp32 = case.get("fp32", False)
    n_pages = (pos + M + PAGE - 1) // PAGE
    pool = _normal(seed, 1, (1, 2, n_pages, kv, PAGE * hd), 1.0, fp32)
    qkv = _normal(seed, 2, (M, (q + 2 * kv) * hd))
    table = torch.randperm(n_pages, generator=_gen(seed, 3), device=DEV).to(torch.int32)
    c, s = sb.rope_table(hd, 10000.0, n_pages * PAGE)
    return pool, qkv, table, torch.from_numpy(c).to(DEV), torch.from_numpy(s).to(DEV)


# ---------------------------------------------------------------- what a program holds before the call
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("projection", "gate_up", "head", "gemm"):
        rows = 2 * case["N"] if kind == "gate_up" else case["N"]
        W = _normal(seed, 1, (rows, case["K"]), 0.02, case.get("fp32", False))
        x = _normal(seed, 2, (case["M"], case["K"]))
        if case.get("kernel", "packed") == "packed":
            W = sb.op_repack(W)
        st = dict(case=case, W=W, x=x)
        if kind == "gemm":
            st["scratch"] = torch.empty(sb.lib().sb_op_gemm_scratch_bytes(rows, case["K"]), dtype=torch.uint8, device=DEV)
        return st
    if kind in ("attention", "prompt_attention"):
        pool, qkv, table, c, s = _attention_inputs(case, seed)
        st = dict(case=case, pool=pool, qkv=qkv, table=table, cos=c, sin=s)
        if kind == "attention":
            n = sb.lib().sb_op_attention_scratch_bytes(case["q"], case["hd"], int(not case["fp32"]), table.numel())
            st["scratch"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        return st

    s, model = _model(case, seed)
    st = dict(case=case, model=model, prompt=_prompt(case, seed))
    if kind == "batch":
        st["sessions"] = [model.session() for _ in range(case["batch"])]
        st["start"], st["script"], st["params"] = [], [], []
        for b, se in enumerate(st["sessions"]):
            p = _prompt(case, seed, b)
            se.prefill(p)
            st["start"].append(len(p))
            st["script"].append(_script(case, seed, b))
            st["params"].append(_params(case, seed + b, st["script"][b]))
        st["sessions"][0].debug_enable()
        st["batch"] = sb.Batch(st["sessions"])
        return st
    se = st["session"] = model.session()
    if kind == "prefill":
        se.kv_pool.zero_()      # (the pool is an output: what the prompt does not reach stays zero)
        se.debug_enable()
        return st
    if kind == "generate":
        fe = _exits(case, seed, case["new"] * case["w"] + 64)
        st["params"] = sb.Params(case["heads"], case["w"], _temps(case["heads"]), 0.5, forced_exit=fe)
        se.debug_enable()
        return st
    first = se.prefill(st["prompt"])
    st["start"] = len(st["prompt"])
    if kind == "decode":
        st["script"] = _script(case, seed)
        st["params"] = _params(case, seed, st["script"])
    else:
        st["first"] = first
        more, _ = se.decode(case["w"], sb.Params(0, 1, [], 2.0))      # the drafts: what greedy decoding would say
        u = np.random.default_rng(seed + 5).random(2 * _capacity(case)).astype(np.float32)
        st["params"] = sb.Params(case["heads"], case["w"], _temps(case["heads"]), 2.0, forced_exit=_exits(case, seed, 64),
                                 forced_draft=np.array(list(more) + [-1] * (64 - len(more)), dtype=np.int32),
                                 sample_temperature=case["temp"], top_p=case["top_p"], sample_u=u)
    se.debug_enable()
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "projection":
        return sb.op_gemv(st["W"], st["x"], PROJ[case["kernel"]])
    if kind == "gate_up":
        return sb.op_gate_up(st["W"], st["x"], PROJ[case["kernel"]])
    if kind == "head":
        am, cf, z = sb.op_head(st["W"], st["x"], case["T"], PROJ[case["kernel"]], want_logits=True)
        return dict(argmax=am, conf=cf, logits=z)
    if kind == "gemm":
        return sb.op_gemm(st["W"], st["x"], st["scratch"])
    if kind == "attention":
        out = sb.op_attention(st["qkv"], case["q"], case["kv"], case["hd"], int(not case["fp32"]), st["pool"], st["table"],
                              0, st["cos"], st["sin"], case["pos"], st["scratch"])
        return dict(out=out, pool=st["pool"])
    if kind == "prompt_attention":
        out = sb.op_prompt_attention(st["qkv"], case["q"], case["kv"], case["hd"], st["pool"], st["table"], 0, st["cos"],
                                     st["sin"], case["pos"])
        return dict(out=out, pool=st["pool"])
    if kind == "batch":
        for r in range(case["rounds"]):
            for se, n, script in zip(st["sessions"], st["start"], st["script"]):
                se.rewind(n + r, script[r], r * case["w"])
            st["batch"].decode(1, st["params"])
        cap = sb.SB_MAX_W // case["batch"]
        return [st["sessions"][0].debug_logits(0, b * cap + i) for b in range(case["batch"]) for i in sorted({0, case["w"] - 1})]
    se = st["session"]
    if kind == "prefill":
        se.prefill(st["prompt"])
        return dict(logits=se.debug_logits(0), kv=se.kv_pool.view(torch.bfloat16))
    if kind == "generate":
        toks, _ = se.generate(st["prompt"], case["new"], st["params"])
        return dict(tokens=toks, logits=se.debug_logits(0))
    if kind == "decode":
        for r in range(case["rounds"]):
            se.rewind(st["start"] + r, st["script"][r], r * case["w"])
            se.decode(1, st["params"])
        return [se.debug_logits(0, i) for i in _rows(case)]
    se.rewind(st["start"], st["first"])
    for _ in range(case["w"]):
        se.draft_step(st["params"])
    v = se.verify(st["params"])
    return dict(n_emit=v["n_emit"], tokens=v["tokens"], prob=np.array(v["accept_prob"], dtype=np.float32),
                logits=se.debug_logits(0, 0))


def _rows(case):
    """Rows of a round whose logits are returned: the first and, where the rows are scripted, the last."""
    return sorted({0, case["w"] - 1}) if case["mode"] == "forced" else [0]


# ---------------------------------------------------------------- what a pass cannot do without
def _layer_flops(s, rows):
    return 2 * rows * (s.layer_weight_bytes() // (2 if s.weight_dtype == si.configs.BF16 else 4))


def _attention_work(q, kv, hd, es, pos, M):
    keys = sum(pos + i + 1 for i in range(M))
    b = 2 * (pos + M) * kv * hd * es + 4 * M * (q + 2 * kv) * hd + 4 * M * q * hd
    return b, 4 * keys * q * hd


def _round_sweeps(exits, L):
    """Layer sweeps (rows of each) and head evaluations of one round with these exit layers."""
    reached, sweeps, heads = [], [], 0
    for e in exits:
        reached.append(0)
        for l in range(1, e + 1):
            rows = [j for j in range(len(reached)) if reached[j] == l - 1 and all(r == l - 1 for r in reached[j:])]
            for j in rows:
                reached[j] = l
            sweeps.append(len(rows))
        heads += e
    top = reached[0]
    for l in range(2, top + 1):
        rows = [j for j in range(len(reached)) if reached[j] == l - 1]
        if rows:
            sweeps.append(len(rows))
            for j in rows:
                reached[j] = l
    return sweeps + [len(exits)] * (L - top), heads


def work(case):
    kind = case["kind"]
    if kind in ("projection", "gate_up", "head", "gemm"):
        N, K, M = case["N"], case["K"], case["M"]
        rows = 2 * N if kind == "gate_up" else N
        return dict(bytes=rows * K * (4 if case.get("fp32") else 2) + 4 * M * (K + N), flops=2 * rows * K * M)
    if kind in ("attention", "prompt_attention"):
        b, f = _attention_work(case["q"], case["kv"], case["hd"], 4 if case.get("fp32") else 2, case["pos"], case["M"])
        return dict(bytes=b, flops=f)
    s = _shape(case)
    lb, hb, L, n = s.layer_weight_bytes(), s.head_weight_bytes(), s.n_layers, case["prompt"]
    es = 2 if s.kv_dtype == si.configs.BF16 else 4
    kvrow = 2 * s.n_kv_heads * s.head_dim * es
    if kind == "prefill":
        f = L * (_layer_flops(s, n) + 4 * (n * (n + 1) // 2) * s.n_heads * s.head_dim) + 2 * s.vocab * s.d_model
        return dict(bytes=L * (lb + n * kvrow) + hb + n * s.d_model * 2 + 4 * s.vocab, flops=f)
    rounds = []
    if kind == "sampled":
        rounds = [_exits(case, 0, case["w"])]
    elif kind == "generate":
        rounds = [_exits(case, r, case["w"]) for r in range(case["new"] - 1)]     # (random heads: a token a round)
    elif case.get("mode") == "forced" or (kind == "batch" and case["w"] > 1):
        rounds = [_exits(case, r, case["w"]) for r in range(case["rounds"])]
    if rounds:
        b = f = 0
        for e in rounds:
            sweeps, heads = _round_sweeps([int(x) for x in e], L)
            b += len(sweeps) * (lb + n * kvrow) + (heads + 1) * hb
            f += sum(_layer_flops(s, m) for m in sweeps) + 2 * (heads + len(e)) * s.vocab * s.d_model
    else:
        B = case.get("batch", 1)
        b = case["rounds"] * (L * (lb + B * n * kvrow) + hb)
        f = case["rounds"] * B * (_layer_flops(s, L) + 2 * s.vocab * s.d_model)
    if kind == "generate":
        b, f = b + L * lb + hb, f + L * _layer_flops(s, n)
    return dict(bytes=b, flops=f)


def tolerance(case):
    """About four times what the paths show against the same in 64 bits."""
    kind = case["kind"]
    if kind in ("projection", "gate_up", "gemm", "head"):
        # fp32 sums over K <= 14080 of bf16 weights times activations that carry 16 mantissa bits: 2.5e-6 to 3.6e-6
        return dict(rel=1.5e-5, max=6e-4, differ=0.0)
    if kind in ("attention", "prompt_attention"):
        # fp32 sums, queries and probabilities as 16-bit pairs: 3e-6 to 6e-6; new keys are rounded to bf16, where a
        # value next to a rounding boundary may fall on the other side (one unit: 2^-8 of it)
        return dict(rel=2e-5, max=1e-2)
    if kind == "generate":
        return dict(rel=1e-6, max=4e-5, differ=0.0)     # fp32 throughout: 2e-7
    # several layers with bf16 keys and values: what the roundings of the cache make of 1e-5 in a projection,
    # 5e-4 to 1.4e-3 after four layers
    return dict(rel=5e-3, max=5e-2, differ=0.0)


# ---------------------------------------------------------------- the same in 64 bits
class _Exact:
    """The decoder in double precision on plain torch, K and V rounded as the cache holds them."""

    def __init__(self, case, seed):
        self.s = _shape(case)
        self.w = _device_weights(case, self.s, seed)
        self.k = [[] for _ in range(self.s.n_layers)]
        self.v = [[] for _ in range(self.s.n_layers)]
        self.n = 0
        hd = self.s.head_dim
        self.inv = (self.s.rope_base ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64) / hd)).to(DEV)

    def _norm(self, x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + self.s.rms_eps) * self.w[g].double()

    def _mm(self, x, name):
        W = self.w[name]
        return torch.cat([x @ c.double().t() for c in W.split(16384)], 1)

    def _rope(self, x, pos):
        a = pos.double()[:, None, None] * self.inv
        h = x.shape[-1] // 2
        c, s = a.cos().float().double(), a.sin().float().double()
        return torch.cat([x[..., :h] * c - x[..., h:] * s, x[..., h:] * c + x[..., :h] * s], -1)

    def _store(self, x):
        return x.to(torch.bfloat16).double() if self.s.kv_dtype == si.configs.BF16 else x.float().double()

    def feed(self, ids):
        """Takes these tokens through all layers; hidden rows after the last one."""
        s = self.s
        T, hq, hkv, hd = len(ids), s.n_heads, s.n_kv_heads, s.head_dim
        pos = torch.arange(self.n, self.n + T, device=DEV)
        h = self.w["embed"][torch.as_tensor(np.asarray(ids, dtype=np.int64), device=DEV)].double()
        for l in range(s.n_layers):
            y = self._mm(self._norm(h, f"attn_norm.{l}"), f"w_qkv.{l}")
            q, k, v = y.split([hq * hd, hkv * hd, hkv * hd], 1)
            q = self._rope(q.view(T, hq, hd), pos)
            self.k[l].append(self._store(self._rope(k.view(T, hkv, hd), pos)))
            self.v[l].append(self._store(v.reshape(T, hkv, hd)))
            K, V = torch.cat(self.k[l]), torch.cat(self.v[l])
            self.k[l], self.v[l] = [K], [V]
            o = _exact_attention(q, K, V, self.n)
            h = h + self._mm(o, f"w_o.{l}")
            g, u = self._mm(self._norm(h, f"ffn_norm.{l}"), f"w_gate_up.{l}").chunk(2, 1)
            h = h + self._mm(g / (1 + torch.exp(-g)) * u, f"w_down.{l}")
        self.n += T
        return h

    def logits(self, h):
        return self._mm(self._norm(h, "final_norm"), "lm_head")

    def scripted(self, prompt, script, case, last):
        """Logits of the rows of the last round: the fed token's and, with `last`, the last draft's."""
        r = case["rounds"]
        h = self.feed(list(prompt) + list(script[:r + case["w"] - 1]))
        at = len(prompt) + r - 1
        return [self.logits(h[at + i:at + i + 1])[0] for i in (sorted({0, case["w"] - 1}) if last else [0])]

    def greedy(self, ids, n):
        """n tokens after ids, and the logits the last one comes from."""
        out = []
        for _ in range(n):
            z = self.logits(self.feed(ids)[-1:])[0]
            out.append(int(z.argmax()))
            ids = out[-1:]
        return out, z


def _exact_attention(q, K, V, pos0):
    """q [T, hq, hd] at positions pos0.. against K, V [n, hkv, hd], causal; [T, hq * hd]."""
    T, hq, hd = q.shape
    G = hq // K.shape[1]
    out = torch.empty_like(q)
    mask = torch.arange(K.shape[0], device=DEV)[None, :] > torch.arange(pos0, pos0 + T, device=DEV)[:, None]
    for i in range(hq):
        z = (q[:, i] @ K[:, i // G].t()) / math.sqrt(hd)
        out[:, i] = torch.softmax(z.masked_fill(mask, -math.inf), 1) @ V[:, i // G]
    return out.reshape(T, hq * hd)


def _pool(K, V, n_pages, table, bf16, base=None):
    """Keys and values [n, hkv, hd] in the paged layout (values of a bf16 pool transposed within a page)."""
    n, hkv, hd = K.shape
    pool = torch.zeros((2, n_pages, hkv, PAGE, hd), dtype=torch.float64, device=DEV) if base is None else base
    pad = n_pages * PAGE - n
    for i, x in enumerate((K, V)):
        pages = torch.cat([x, x.new_zeros(pad, hkv, hd)]).view(n_pages, PAGE, hkv, hd).permute(0, 2, 1, 3)
        pages = pages.transpose(2, 3).reshape(n_pages, hkv, PAGE, hd) if i == 1 and bf16 else pages
        pool[i][table.long()] = pages
    return pool


def exact(case, seed):
    kind = case["kind"]
    if kind in ("projection", "gate_up", "head", "gemm"):
        rows = 2 * case["N"] if kind == "gate_up" else case["N"]
        W = _normal(seed, 1, (rows, case["K"]), 0.02, case.get("fp32", False))
        x = _normal(seed, 2, (case["M"], case["K"])).double()
        z = torch.cat([x @ c.double().t() for c in W.split(16384)], 1)
        if kind == "gate_up":
            g, u = z.chunk(2, 1)
            return g / (1 + torch.exp(-g)) * u
        if kind == "head":
            top = z.max(1, keepdim=True)
            conf = 1.0 / torch.exp((z - top.values) / case["T"]).sum(1)
            return dict(argmax=top.indices[:, 0].to(torch.int32), conf=conf, logits=z)
        return z
    if kind in ("attention", "prompt_attention"):
        hd, kv, q, M, pos = case["hd"], case["kv"], case["q"], case["M"], case["pos"]
        fp32 = case.get("fp32", False)
        pool, qkv, table, c, s = _attention_inputs(case, seed)
        n_pages, n = table.numel(), pos + M
        P = pool.view(2, n_pages, kv, PAGE * hd).double()[:, table.long()]     # logical pages
        K = P[0].view(n_pages, kv, PAGE, hd).permute(0, 2, 1, 3).reshape(-1, kv, hd)[:n].clone()
        V = P[1].view(n_pages, kv, PAGE, hd) if fp32 else P[1].view(n_pages, kv, hd, PAGE).transpose(2, 3)
        V = V.permute(0, 2, 1, 3).reshape(-1, kv, hd)[:n].clone()
        x, k, v = qkv.double().split([q * hd, kv * hd, kv * hd], 1)
        cos, sin = c[pos:n].double()[:, None], s[pos:n].double()[:, None]

        def rope(t):
            a, b = t[..., :hd // 2], t[..., hd // 2:]
            return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

        def store(t):
            return t if fp32 else t.to(torch.bfloat16).double()

        K[pos:], V[pos:] = store(rope(k.view(M, kv, hd))), store(v.reshape(M, kv, hd))
        out = _exact_attention(rope(x.view(M, q, hd)), K, V, pos)
        # (slots past the last key: not written by the fp32 kernel, zeroed or left by the bf16 ones -- no value)
        whole = n % PAGE == 0
        return dict(out=out, pool=_pool(K, V, n_pages, table, not fp32).view(pool.shape) if whole else None)
    if kind == "batch":
        return [z for b in range(case["batch"])
                for z in _Exact(case, seed).scripted(_prompt(case, seed, b), _script(case, seed, b), case, True)]
    m = _Exact(case, seed)
    prompt = list(_prompt(case, seed))
    if kind == "prefill":
        z = m.logits(m.feed(prompt)[-1:])[0]
        pages = _capacity(case) // PAGE
        table = torch.arange(pages, device=DEV)
        kv = torch.stack([_pool(m.k[l][0], m.v[l][0], pages, table, True) for l in range(m.s.n_layers)])
        return dict(logits=z, kv=kv.reshape(-1))
    if kind == "generate":
        t, z = m.greedy(prompt, case["new"])
        return dict(tokens=torch.tensor(t, dtype=torch.int32), logits=z)
    if kind == "decode":
        return m.scripted(prompt, _script(case, seed), case, case["mode"] == "forced")
    t, _ = m.greedy(prompt, 1)
    z = m.logits(m.feed(t))[0]
    return dict(n_emit=None, tokens=[None] * case["w"], prob=None, logits=z)
