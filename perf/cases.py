"""Workloads of the pipeline-stage executor, as data: what a serving program has a stage do,
from one short question on a single sequence to the largest prompt pass, in both directions of
generation (prompt pass, generation step), both storage types, with and without the LM head,
and with the weights resident or still arriving from host memory.

A case is one call (or one short generation) of `Stage`.  Shapes are this package's own
configurations (`synth.CONFIGS`); a stage holds one or two layers of them, enough that its
weights do not stay in the chip's 256 MB cache from one pass to the next, so that a generation
step streams them from memory as it does inside a whole model.

Keys of a case
  kind    "prompt" (one prompt pass), "step" (one generation step on filled caches),
          "generate" (prompt pass, then `steps` generation steps), "stream" (blocks are copied
          from pinned host memory while the prompt pass runs behind them)
  model   a key of synth.CONFIGS;  dtype: storage type (the configuration's own, or "f32")
  layers  layers the stage holds;  head: it also holds the final norm and the LM head and
          returns logits;  steps: generation steps of "generate"
  batch   sequences;  lo, hi: prompt lengths ("prompt", "generate", "stream") or cached
          context lengths ("step") are spread over [lo, hi]
"""
import math
import random

import torch

import synth
from paper_2502_09922_amd import Stage, binding

C = binding.C


def listed():
    return [
        # the smallest call: the tiny fp32 model as a whole, a 32-token prompt and 8 tokens
        # after it; nothing but latency and launches
        dict(name="tiny_f32_generate", kind="generate", model="tiny_f32", dtype="f32", layers=2, head=True, batch=1,
             lo=32, hi=32, steps=8),
        # fp32 storage at a real layer size, as one checks a bf16 deployment against it
        dict(name="7b_f32_prompt", kind="prompt", model="llama7b", dtype="f32", layers=1, head=False, batch=2, lo=131,
             hi=190),
        # one short question: fewer rows than the prompt GEMM's tile
        dict(name="7b_prompt_1x45", kind="prompt", model="llama7b", dtype="bf16", layers=2, head=False, batch=1, lo=45,
             hi=45),
        # one ordinary prompt on its own (time to first token of an interactive request)
        dict(name="7b_prompt_1x311", kind="prompt", model="llama7b", dtype="bf16", layers=2, head=False, batch=1, lo=311,
             hi=311),
        # the largest: the 13B-shaped benchmark's prompt pass, 32 x 1024 tokens
        dict(name="13b_prompt_32x1024", kind="prompt", model="llama13b", dtype="bf16", layers=1, head=False, batch=32,
             lo=1024, hi=1024),
        # grouped-query model, ragged prompts packed without padding
        dict(name="70b_prompt_ragged", kind="prompt", model="llama70b", dtype="bf16", layers=1, head=False, batch=6,
             lo=128, hi=2048),
        # execute-while-load: two layer blocks arrive over the host link under an 8 x 512 prompt pass
        dict(name="7b_stream_8x512", kind="stream", model="llama7b", dtype="bf16", layers=2, head=False, batch=8, lo=512,
             hi=512),
        # one interactive sequence with a long context
        dict(name="7b_step_b1", kind="step", model="llama7b", dtype="bf16", layers=2, head=False, batch=1, lo=3000,
             hi=3000),
        # the last stage of a small deployment: layer, final norm, LM head, logits
        dict(name="7b_step_b8_head", kind="step", model="llama7b", dtype="bf16", layers=1, head=True, batch=8, lo=512,
             hi=640),
        # the 13B-shaped benchmark's generation step
        dict(name="13b_step_b32", kind="step", model="llama13b", dtype="bf16", layers=2, head=False, batch=32, lo=1024,
             hi=1087),
        # the 70B-shaped benchmark's: ragged contexts, grouped queries
        dict(name="70b_step_b64_ragged", kind="step", model="llama70b", dtype="bf16", layers=2, head=False, batch=64,
             lo=128, hi=2287),
        # a full server: more sequences than one weight-streaming pass takes
        dict(name="13b_step_b100", kind="step", model="llama13b", dtype="bf16", layers=2, head=False, batch=100, lo=64,
             hi=900),
    ]


# ---- sizes ---------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _params(s):
    """Weights of one decoder layer."""
    return s.qkv_rows * s.hidden + s.hidden * s.n_q_heads * s.head_dim + 3 * s.ffn * s.hidden + 2 * s.hidden


def draw(rng):
    kind = rng.choice(["prompt"] * 9 + ["step"] * 9 + ["generate", "stream"])
    if kind == "generate":
        lo = _log_int(rng, 4, 100)
        return dict(kind=kind, model="tiny_f32", dtype="f32", layers=2, head=True, batch=rng.randint(1, 4), lo=lo,
                    hi=lo + rng.randint(0, 28), steps=rng.randint(2, 12))
    f32 = kind != "stream" and rng.random() < 0.12
    model = "llama7b" if f32 or kind == "stream" else rng.choice(["llama7b", "llama13b", "llama70b"])
    head = kind != "stream" and rng.random() < 0.2
    case = dict(kind=kind, model=model, dtype="f32" if f32 else "bf16", head=head)
    if kind == "step":
        hi = _log_int(rng, 64, 512 if f32 else 4096)
        # caches of at most 200k positions (64k for the multi-head models), at most 128 sequences
        room = (200_000 if model == "llama70b" else 64_000) // hi
        case.update(layers=1 if f32 or head else 2, batch=_log_int(rng, 1, min(32 if f32 else 128, max(1, room))),
                    lo=max(16, int(hi * rng.uniform(0.1, 1.0))), hi=hi)
        return case
    # prompts of 16..2048 tokens, at most 512 rows in fp32 and never more work than 32 x 1024 rows
    # of the 13B-shaped layer
    shape, big = synth.CONFIGS[model], synth.CONFIGS["llama13b"]
    most = 512 if f32 else int(0.95 * 32768 * _params(big) / _params(shape))
    rows = _log_int(rng, 16, min(most, 8192 if kind == "stream" else most))
    batch = min(_log_int(rng, 1, 32), max(1, rows // 16))
    hi = min(2048, max(16, rows // batch))
    case.update(layers=2 if kind == "stream" or batch * hi < 2048 and not f32 and not head else 1, batch=batch,
                lo=max(8, int(hi * rng.choice([1.0, rng.uniform(0.2, 1.0)]))), hi=hi)
    return case


def _lengths(case):
    """Lengths of the batch's sequences: `hi` first, the others spread over [lo, hi]."""
    r = random.Random("%d %d %d" % (case["batch"], case["lo"], case["hi"]))
    return [case["hi"]] + [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"] - 1)]


def _shape(case):
    """The model the stage belongs to: a middle stage of it (no embedding, no head), its last
    stage, or (tiny model) the whole of it."""
    s = synth.CONFIGS[case["model"]].with_(dtype=case["dtype"])
    if case["kind"] == "generate":
        return s, 0, s.n_layers_total
    s = s.with_(n_layers_total=case["layers"] + 1)
    return (s if case["head"] else s.with_(vocab=0)), 1, case["layers"] + 1


def _max_seq(case):
    return (case["hi"] + case.get("steps", 1) + 255) // 256 * 256


# ---- values ----------------------------------------------------------------------------------
# Matrices N(0, 0.02), gains 1 + N(0, 0.02), hidden inputs N(0, 1), token ids uniform: the
# recipe of synth/gen.py, drawn on the device.  A tensor depends on the seed and its own name only.
def _gen(seed, *key):
    return torch.Generator(device="cuda").manual_seed(random.Random("%d %r" % (seed, key)).randrange(1 << 62))


def _normal(seed, key, size, dtype, mean=0.0, std=1.0):
    out = torch.empty(size, dtype=dtype, device="cuda")
    return out.normal_(mean, std, generator=_gen(seed, *key))


def _block(s, seed, layer):
    """The tensors of one block, in block order."""
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    d, qd = s.hidden, s.n_q_heads * s.head_dim
    if layer == -1:
        sizes = [("embed", (s.vocab, d))]
    elif layer == s.n_layers_total:
        sizes = [("final_norm", (d,)), ("lm_head", (s.vocab, d))]
    else:
        sizes = [("attn_norm", (d,)), ("wqkv", (s.qkv_rows, d)), ("wo", (d, qd)), ("ffn_norm", (d,)),
                 ("wgu", (2 * s.ffn, d)), ("wd", (d, s.ffn))]
    return [_normal(seed, (layer, n), z, dt, 1.0 if n.endswith("norm") else 0.0, 0.02) for n, z in sizes]


def _inputs(case, s, seed):
    """Inputs of the calls of one pass, in order."""
    lens = _lengths(case)
    rows = case["batch"] if case["kind"] == "step" else sum(lens)
    if case["kind"] == "generate":
        return [torch.randint(0, s.vocab, (rows if t == 0 else case["batch"],), dtype=torch.int32, device="cuda",
                              generator=_gen(seed, "tokens", t)) for t in range(case["steps"] + 1)]
    return [_normal(seed, ("hidden",), (rows, s.hidden), torch.float32 if s.dtype == "f32" else torch.bfloat16)]


def _caches(case, s, seed, lo, hi):
    """Filled key and value caches of a generation step: keys and values of such a model are sums
    of `hidden` products of a normalised row and N(0, 0.02) weights."""
    size = (hi - lo, case["batch"], s.n_kv_heads, _max_seq(case), s.head_dim)
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    std = 0.02 * math.sqrt(s.hidden)
    return _normal(seed, ("k",), size, dt, 0.0, std), _normal(seed, ("v",), size, dt, 0.0, std)


# ---- the package's side -------------------------------------------------------------------------
def prepare(case, seed):
    s, lo, hi = _shape(case)
    lens = _lengths(case)
    rows = case["batch"] if case["kind"] == "step" else sum(lens)
    st = Stage(s, lo, hi, case["batch"], _max_seq(case), rows)
    host = {}
    for layer in st.block_ids():
        view = st.block_view(layer)
        off, nb = C.c_size_t(), C.c_size_t()
        for i, t in enumerate(_block(s, seed, layer)):
            binding.check(binding.lib.ls_block_tensor(C.byref(st.cfg), layer, i, C.byref(off), C.byref(nb)))
            view[off.value : off.value + nb.value].view(t.dtype).copy_(t.view(-1))
        if case["kind"] == "stream":
            host[layer] = torch.empty(view.numel(), dtype=torch.uint8, pin_memory=True)
            host[layer].copy_(view)
        else:
            st.adopt_block(layer)
    size = (hi - lo, case["batch"], s.n_kv_heads, _max_seq(case), s.head_dim)
    state = dict(case=case, stage=st, host=host, lens=lens, inputs=_inputs(case, s, seed),
                 k=st.k.view(st.tdtype).view(size), v=st.v.view(st.tdtype).view(size))
    if case["kind"] == "step":
        k, v = _caches(case, s, seed, lo, hi)
        state["k"].copy_(k)
        state["v"].copy_(v)
        state["ctx"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    if case["kind"] == "stream":
        st.slab.zero_()
        state["copies"] = torch.cuda.Stream()
    torch.cuda.synchronize()
    return state


def run(state):
    case, st, lens, inputs = state["case"], state["stage"], state["lens"], state["inputs"]
    head = case["head"]
    outs = []
    if case["kind"] == "step":
        # the scheduler names the cached length of every slot, then the step runs
        st.seq_lens.copy_(state["ctx"])
        outs.append(st.decode(inputs[0], case["batch"], case["hi"], want_logits=head))
    else:
        if case["kind"] == "stream":
            st.reset_blocks()
            state["copies"].wait_stream(torch.cuda.current_stream())  # the last pass is done with the slab
            for layer in st.block_ids():
                st.load_block(layer, state["host"][layer], state["copies"])
        outs.append(st.prefill(inputs[0], lens, want_logits=head))
        for t in range(case.get("steps", 0)):
            outs.append(st.decode(inputs[1 + t], case["batch"], case["hi"] + t, want_logits=head))
    # with a head: logits (the next token is their largest entry, a rounding away from the
    # second one now and then); without: hidden states.  The caches are updated state.
    return {"out": [o[1] if head else o for o in outs], "k": state["k"], "v": state["v"], "seq_lens": st.seq_lens}


# ---- what a pass cannot do without ---------------------------------------------------------------
def work(case):
    s, lo, hi = _shape(case)
    e, lens, n = s.itemsize, _lengths(case), hi - lo
    kv_row = 2 * s.n_kv_heads * s.head_dim * e  # key and value of one position of one layer
    head = (s.vocab * s.hidden + s.hidden) if case["head"] else 0

    def one(rows, batch, reads, pairs):
        """rows through the stage, `reads` cached positions read, `pairs` (query, key) pairs a head."""
        flops = 2.0 * rows * n * _params(s) + 4.0 * n * s.n_q_heads * s.head_dim * pairs + 2.0 * batch * head
        move = (n * _params(s) + head) * e + n * kv_row * (reads + rows)
        move += rows * (4 if case["kind"] == "generate" else s.hidden * e) + (4 * batch * s.vocab if head else rows * s.hidden * e)
        return flops, float(move)

    if case["kind"] == "step":
        calls = [one(case["batch"], case["batch"], sum(lens), sum(l + 1 for l in lens))]
    else:
        calls = [one(sum(lens), case["batch"], 0, sum(l * (l + 1) // 2 for l in lens))]
        calls += [one(case["batch"], case["batch"], sum(lens) + case["batch"] * t, sum(l + t + 1 for l in lens))
                  for t in range(case.get("steps", 0))]
    return {"bytes": sum(c[1] for c in calls), "flops": sum(c[0] for c in calls)}


def tolerance(case):
    # Measured against `exact`: fp32 2.8e-6 (sums of up to 11008 products); bf16 4e-3..8e-3 at the 7B
    # and 13B shapes and 1.1e-2 at the 70B shape, after one or two layers (normalised rows, q/k/v,
    # softmax weights, attention output and SwiGLU output are rounded to 8 bits on their way, and
    # every layer amplifies the differences of the one before).
    return {"rel": 1e-5, "max": 4e-4} if case["dtype"] == "f32" else {"rel": 2e-2, "max": 0.2}


# ---- the same in 64 bits, plain torch ---------------------------------------------------------
def exact(case, seed):
    s, lo, hi = _shape(case)
    lens, inputs = _lengths(case), _inputs(case, s, seed)
    B, G, hd, f64 = case["batch"], s.n_q_heads // s.n_kv_heads, s.head_dim, torch.float64
    if case["kind"] == "step":
        k, v = (t.double() for t in _caches(case, s, seed, lo, hi))
    else:
        k = torch.zeros(hi - lo, B, s.n_kv_heads, _max_seq(case), hd, dtype=f64, device="cuda")
        v = torch.zeros_like(k)
    freq = s.rope_base ** (-2.0 * torch.arange(hd // 2, dtype=f64, device="cuda") / hd)

    def norm(x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + float(torch.tensor(s.rms_eps, dtype=torch.float32))) * g.double()

    def turn(t, pos):  # [rows, heads, hd], pairs (2i, 2i + 1)
        a = pos.double()[:, None] * freq
        c, n = torch.cos(a)[:, None], torch.sin(a)[:, None]
        u, w = t[..., 0::2], t[..., 1::2]
        return torch.stack([u * c - w * n, u * n + w * c], -1).reshape(t.shape)

    def call(inp, news, olds):
        """One call: sequence b brings news[b] rows behind olds[b] cached positions."""
        if case["kind"] == "generate":
            x = _block(s, seed, -1)[0][inp.long()].double()
        else:
            x = inp.double()
        pos = torch.cat([torch.arange(o, o + n, device="cuda") for n, o in zip(news, olds)])
        for li in range(hi - lo):
            g1, wqkv, wo, g2, wgu, wd = _block(s, seed, lo + li)
            qkv = (norm(x, g1) @ wqkv.double().t()).view(-1, s.n_q_heads + 2 * s.n_kv_heads, hd)
            q = turn(qkv[:, : s.n_q_heads], pos)
            kn = turn(qkv[:, s.n_q_heads : s.n_q_heads + s.n_kv_heads], pos)
            vn = qkv[:, s.n_q_heads + s.n_kv_heads :]
            att, r = torch.empty(x.shape[0], s.n_q_heads, hd, dtype=f64, device="cuda"), 0
            for b, (n, o) in enumerate(zip(news, olds)):
                k[li, b, :, o : o + n] = kn[r : r + n].transpose(0, 1)
                v[li, b, :, o : o + n] = vn[r : r + n].transpose(0, 1)
                keys, vals = k[li, b, :, : o + n].contiguous(), v[li, b, :, : o + n].contiguous()
                qb = q[r : r + n].view(n, s.n_kv_heads, G, hd).permute(1, 2, 0, 3).reshape(s.n_kv_heads, G * n, hd)
                sc = torch.bmm(qb, keys.transpose(1, 2).contiguous()).view(s.n_kv_heads, G, n, o + n) / math.sqrt(hd)
                seen = torch.arange(o + n, device="cuda")[None] <= (o + torch.arange(n, device="cuda"))[:, None]
                p = torch.softmax(sc.masked_fill(~seen, -math.inf), -1).view(s.n_kv_heads, G * n, o + n)
                ob = torch.bmm(p, vals).view(s.n_kv_heads, G, n, hd).permute(2, 0, 1, 3)
                att[r : r + n] = ob.reshape(n, s.n_q_heads, hd)
                r += n
            x = x + att.view(x.shape[0], -1) @ wo.double().t()
            gu = norm(x, g2) @ wgu.double().t()
            x = x + (torch.nn.functional.silu(gu[:, : s.ffn]) * gu[:, s.ffn :]) @ wd.double().t()
        if not case["head"]:
            return x
        g, w = _block(s, seed, s.n_layers_total)
        last = torch.cumsum(torch.tensor(news, device="cuda"), 0) - 1
        return norm(x[last], g) @ w.double().t()

    if case["kind"] == "step":
        outs, total = [call(inputs[0], [1] * B, lens)], [l + 1 for l in lens]
    else:
        outs, total = [call(inputs[0], lens, [0] * B)], list(lens)
        for t in range(case.get("steps", 0)):
            outs.append(call(inputs[1 + t], [1] * B, total))
            total = [l + 1 for l in total]
    return {"out": outs, "k": k, "v": v, "seq_lens": torch.tensor(total, dtype=torch.int32, device="cuda")}
