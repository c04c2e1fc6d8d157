"""Models of few layers whose matrices are wide enough for the launches that the tiny models never reach, against the same layers in
double precision on plain torch (the CPU oracle would take minutes)."""
import math

import numpy as np
import pytest

import sb_inputs as si
from helpers import gpu_model

pytestmark = pytest.mark.gpu

B16, F32 = si.configs.BF16, si.configs.FP32


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    return torch


def _weights(T, shape, seed):
    """({name: host array}, {name: GPU tensor}), all layers of the same matrices, norm gains jittered."""
    g = T.Generator(device="cuda")
    g.manual_seed(seed)
    dev = {}
    for name, shp, std in si.tensor_specs(shape):
        base = name.split(".")[0]
        first = f"{base}.0"
        if name != first and first in dev:
            dev[name] = dev[first]
        else:
            dev[name] = (T.randn(shp, generator=g, device="cuda") * std).to(T.bfloat16)
    for name in ["final_norm"] + [f"{n}.{l}" for l in range(shape.n_layers) for n in ("attn_norm", "ffn_norm")] + \
            [f"exit_norm.{l}" for l in range(shape.n_exit_heads)]:
        dev[name] = 1.0 + 0.1 * T.randn(shape.d_model, generator=g, device="cuda")
    host = {}
    for name, t in dev.items():
        same = next((n for n in host if dev[n] is t), None)
        host[name] = host[same] if same else (t.cpu().view(T.int16).numpy().view(np.uint16) if t.dtype == T.bfloat16 else t.cpu().numpy())
    return host, dev


def _double(T, shape, w, ids, upto):
    """(rotated keys, values of layer `upto`), or the logits of every row where upto == n_layers."""
    hd, hq, hkv = shape.head_dim, shape.n_heads, shape.n_kv_heads
    n = len(ids)
    inv = shape.rope_base ** (-2.0 * T.arange(hd // 2, dtype=T.float64, device="cuda") / hd)
    ang = T.arange(n, device="cuda").double()[:, None, None] * inv
    c, s = ang.cos().float().double(), ang.sin().float().double()

    def norm(x, g):
        return x / T.sqrt((x * x).mean(-1, keepdim=True) + shape.rms_eps) * w[g].double()

    def mm(x, name):
        return T.cat([x @ p.double().t().contiguous() for p in w[name].split(8192)], 1)

    def rope(x):
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return T.cat([a * c - b * s, b * c + a * s], -1)

    h = w["embed"][T.as_tensor(np.asarray(ids, dtype=np.int64), device="cuda")].double()
    mask = T.ones(n, n, dtype=T.bool, device="cuda").triu(1)
    for l in range(shape.n_layers):
        q, k, v = mm(norm(h, f"attn_norm.{l}"), f"w_qkv.{l}").split([hq * hd, hkv * hd, hkv * hd], 1)
        q, k, v = rope(q.view(n, hq, hd)), rope(k.view(n, hkv, hd)), v.reshape(n, hkv, hd)
        if l == upto:
            return k.reshape(n, -1).cpu().numpy(), v.reshape(n, -1).cpu().numpy()
        o = T.empty_like(q)
        for i in range(hq):
            z = (q[:, i] @ k[:, i * hkv // hq].t().contiguous()) / math.sqrt(hd)
            o[:, i] = T.softmax(z.masked_fill(mask, -math.inf), 1) @ v[:, i * hkv // hq].contiguous()
        h = h + mm(o.reshape(n, -1), f"w_o.{l}")
        a, b = mm(norm(h, f"ffn_norm.{l}"), f"w_gate_up.{l}").chunk(2, 1)
        h = h + mm(a / (1 + T.exp(-a)) * b, f"w_down.{l}")
    return mm(norm(h, "final_norm"), "lm_head").cpu().numpy()


def _worst_kv(session, ref, layer):
    """Largest error of a position's keys and values, as a share of its largest."""
    worst = 0.0
    for pos in range(len(ref[0])):
        for got, want in zip(session.debug_kv(layer, pos), (ref[0][pos], ref[1][pos])):
            worst = max(worst, float(np.max(np.abs(got - want)) / np.max(np.abs(want))))
    return worst


# 512 rows in passes of 128: 256, 512, 768 and 1024 attention blocks (a chip full) of both head sizes; 1100 rows: up to 2048
@pytest.mark.parametrize("Hq,Hkv,hd,n", [(32, 8, 64, 512), (16, 16, 128, 512), (16, 16, 128, 1100)])
def test_prompt_through_fp32_cache_block_counts(T, Hq, Hkv, hd, n):
    shape = si.tiny_shape(n_layers=2, n_exit_heads=1, weight_dtype=B16, kv_dtype=F32, d_model=2048, n_heads=Hq, n_kv_heads=Hkv, head_dim=hd,
                          d_ffn=768)
    host, dev = _weights(T, shape, 5 + hd)
    prompt = si.make_prompt(shape.vocab, n, 7)
    s = gpu_model(shape, host, 1120).session()
    s.prefill(prompt)
    # five products in a row, each within 3e-5 of its largest value, between norms that keep the scale
    assert _worst_kv(s, _double(T, shape, dev, prompt, 1), 1) <= 1.5e-4


# gate / up of a single pass in ranges of 9 k blocks (weights requested a whole block at a time) and of 10 (step by step), 8 k blocks a row
# block: a range begins and ends inside one, and some row blocks are finished by the GEMM, others by its epilogue
@pytest.mark.parametrize("d_ffn", [36096, 38400])
def test_prompt_gate_up_ranges(T, d_ffn):
    shape = si.tiny_shape(n_layers=2, n_exit_heads=1, weight_dtype=B16, kv_dtype=F32, d_model=1024, n_heads=8, n_kv_heads=8, head_dim=128,
                          d_ffn=d_ffn)
    host, dev = _weights(T, shape, d_ffn)
    m = gpu_model(shape, host, 160)
    for n in (9, 20, 45, 63, 80, 96, 97, 128):   # (every number of column tiles)
        prompt = si.make_prompt(shape.vocab, n, 11 + n)
        s = m.session()
        s.prefill(prompt)
        worst = _worst_kv(s, _double(T, shape, dev, prompt, 1), 1)
        assert worst <= 1.5e-4, (n, worst)


def _wide_model(T):
    """4224 x 4224 and 4224 x 12416 projections onto the hidden row (two tiles per block), 7040 rows of Q K V, gate / up in two pairs per block."""
    shape = si.tiny_shape(n_layers=3, n_exit_heads=2, weight_dtype=B16, kv_dtype=F32, d_model=4224, n_heads=33, n_kv_heads=11, head_dim=128,
                          d_ffn=12416, vocab=1024)
    return (shape, *_weights(T, shape, 21))


def _script(n, seed):
    return np.random.default_rng(seed).integers(0, 1024, n).astype(np.int32)


def _rounds(sb, script, rounds, w, exits):
    """Params of rounds that start at a token of the script and draft the ones after it."""
    fd = np.concatenate([script[r + 1:r + 1 + w] for r in range(rounds)])
    return sb.Params(2, w, [2.0, 1.0], 2.0, forced_exit=np.resize(exits, len(fd)).astype(np.int32), forced_draft=fd)


@pytest.mark.parametrize("proj", ["mfma_packed", "mfma", "valu"])
def test_wide_decode_rounds(T, proj):
    """Passes of one to eight rows through projections of every block shape above 4096 rows, with the residual and its sums of squares."""
    import paper_2604_12247_amd as sb
    shape, host, dev = _wide_model(T)
    m = gpu_model(shape, host, 96, {"mfma_packed": sb.PROJ_MFMA_PACKED, "mfma": sb.PROJ_MFMA, "valu": sb.PROJ_VALU}[proj])
    prompt = si.make_prompt(shape.vocab, 21, 3)
    for w in (1, 2, 3, 6, 8):
        s = m.session()
        s.prefill(prompt)
        s.debug_enable()
        script = _script(3 + w, w)
        p = _rounds(sb, script, 3, w, [1, 2, 2])
        for r in range(3):
            s.rewind(len(prompt) + r, script[r], r * w)
            s.decode(1, p)
        ref = _double(T, shape, dev, list(prompt) + list(script[:w + 2]), shape.n_layers)
        for i in range(w):
            want = ref[len(prompt) + 2 + i]
            # three layers of five products, each within 3e-5 of its largest value (1e-5 each on the vector ALU)
            assert np.max(np.abs(s.debug_logits(0, i) - want)) <= 4.5e-4 * np.max(np.abs(want)), (w, i)


@pytest.mark.parametrize("B,w", [(4, 2), (4, 1), (3, 2), (2, 4)])
def test_wide_batch_equals_each_sequence_alone(T, B, w):
    """Sweeps that gather one to all of the sequences (they leave the early layers at different exits): every row's logits are, bit for
    bit, those of its sequence alone."""
    import paper_2604_12247_amd as sb
    shape, host, _ = _wide_model(T)
    m = gpu_model(shape, host, 96)
    prompts = [si.make_prompt(shape.vocab, 12 + 5 * b, 40 + b) for b in range(B)]
    scripts = [_script(4 + w, 60 + b) for b in range(B)]
    P = [_rounds(sb, scripts[b], 4, w, [[1, 2], [2], [1], [2, 1, 1]][b]) for b in range(B)]
    alone = []
    for b in range(B):
        s = m.session()
        s.prefill(prompts[b])
        s.debug_enable()
        for r in range(4):
            s.rewind(len(prompts[b]) + r, scripts[b][r], r * w)
            s.decode(1, P[b])
        alone.append([s.debug_logits(0, i) for i in range(w)])
    sess = [m.session() for _ in range(B)]
    for s, p in zip(sess, prompts):
        s.prefill(p)
    sess[0].debug_enable()
    bt, cap = sb.Batch(sess), sb.SB_MAX_W // B
    for r in range(4):
        for s, p, script in zip(sess, prompts, scripts):
            s.rewind(len(p) + r, script[r], r * w)
        bt.decode(1, P)
    for b in range(B):
        for i in range(w):
            assert np.array_equal(sess[0].debug_logits(0, b * cap + i), alone[b][i]), (b, i)
