"""The work that a VLM post-training program has this framework do, as timed cases.

Every case is one call (the fp32 one two) of ``runtime.DeviceModel`` on one GPU:

* ``prefix``: the prompt prefill over visual and text tokens;
* ``suffix``: scoring sampled responses against the kept prefix KV, per prompt or with the
  prompt's KV shared by a group of responses;
* ``prompt``: scoring the prompts' own text tokens from the prefix pass's hidden state;
* ``decode``: one rollout step of a batch, from its KV cache;
* ``both``: prefix then suffix of the fp32 model.

Models are the repository's own slices (``configs.py``): the 7B- and 32B-shaped backbones in
bf16 or fp16 and the tiny fp32 one.  Weights are N(0, 0.02) with norm weights around 1 and
q/k/v biases; visual embeddings N(0, 1); ids uniform.  Keys, values and boundary states that a
call takes from an earlier pass have the spread that such a pass leaves (a projection of a
normed row by N(0, 0.02) weights: about 0.02 sqrt(d)).
"""
from __future__ import annotations

import math
import zlib
from dataclasses import replace

import torch

from paper_2608_14498_amd import binding as rb
from paper_2608_14498_amd.configs import QWEN32B_SLICE, QWEN7B_SLICE, TINY, ModelShape
from paper_2608_14498_amd.runtime import DeviceModel

MODELS = {"tiny": TINY, "7b": QWEN7B_SLICE, "32b": QWEN32B_SLICE}
MAX_POSITION = 32768
TEXT_SHARE = 0.08  # of a prompt; the rest are visual slots


# ------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------
def listed():
    return [
        # the tail of a rollout: one straggler still decodes, so every weight is read for one row
        dict(name="decode_b1_kv4000", kind="decode", model="7b", dtype="bf16", layers=4, batch=1, kv_lo=4000, kv_hi=4000),
        # the repository's co-location rollout: 64 sequences over an 8192-token cache
        dict(name="decode_b64_kv8192", kind="decode", model="7b", dtype="bf16", layers=4, batch=64, kv_lo=8192, kv_hi=8192),
        # a full rollout batch (20 prompts x 8 responses) of short video prompts at mixed lengths
        dict(name="decode_b160_kv500_3000", kind="decode", model="7b", dtype="bf16", layers=4, batch=160, kv_lo=500, kv_hi=3000),
        # one prompt of the smallest median length of the video tasks (470 tokens), as it arrives
        dict(name="prefix_p470", kind="prefix", model="7b", dtype="bf16", layers=1, lens="470", mrope=True, last_rows=False),
        # a small batch of ordinary prompts of mixed lengths, multimodal positions, every row's
        # final hidden state kept (for scoring the prompts)
        dict(name="prefix_ragged_b4", kind="prefix", model="7b", dtype="bf16", layers=1, lens="5900,1733,4096,2500", mrope=True, last_rows=False, hidden=True),
        # the headline workload's prefill: 2 x 16384 tokens, 32B-shaped layers (a whole call)
        dict(name="prefix_32b_2x16384", kind="prefix", model="32b", dtype="bf16", layers=2, lens="16384,16384", mrope=False, last_rows=False),
        # a prefill that only feeds the suffix pass (last layer at the boundary rows), fp16 storage
        dict(name="prefix_last_rows_f16", kind="prefix", model="7b", dtype="f16", layers=2, lens="2048,3001,1200", mrope=True, last_rows=True),
        # one short response scored against its prompt, as it finishes
        dict(name="suffix_s48", kind="suffix", model="7b", dtype="bf16", layers=1, prefix="1501", group=1, lens="48", fused=False),
        # the repository's 7B scoring batch: 4 responses of 256 tokens over 4096-token prompts (a whole call)
        dict(name="suffix_b4_s256", kind="suffix", model="7b", dtype="bf16", layers=4, prefix="4096,4096,4096,4096", group=1, lens="256,256,256,256", fused=False),
        # GRPO groups: 2 prompts x 8 responses of mixed lengths sharing each prompt's KV, no stored logits
        dict(name="suffix_grpo_2x8", kind="suffix", model="7b", dtype="bf16", layers=1, prefix="4096,8190", group=8,
             lens="256,700,431,64,512,333,1000,129,256,870,90,512,401,256,640,77", fused=True),
        # prompt text tokens of a batch scored from the kept hidden state
        dict(name="prompt_r600", kind="prompt", model="7b", dtype="bf16", layers=1, lens="4096,3500", rows=600, fused=False),
        # the fp32 model: both passes over 2 x 512 prompt tokens and 2 x 64 response tokens
        dict(name="tiny_f32_b2", kind="both", model="tiny", dtype="f32", layers=2, prefix="512,512", lens="64,64"),
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _texts(v):
    return ",".join(str(int(x)) for x in v)


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefix", "prefix", "suffix", "suffix", "suffix", "prompt", "both"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    if kind == "decode":
        batch = _spread(rng, 1, 192)
        hi = _spread(rng, 256, min(16384, 600000 // batch))
        return dict(kind="decode", model="7b", dtype=dtype, layers=rng.choice([1, 4]), batch=batch, kv_lo=rng.randint(max(1, hi // 4), hi), kv_hi=hi)
    if kind == "prefix":
        model = rng.choice(["7b", "7b", "32b"])
        total, lens = _spread(rng, 100, 24000), []
        while total >= 64 and len(lens) < 8:
            n = min(total, 12288, _spread(rng, 64, max(65, total)))
            lens.append(n)
            total -= n
        last = rng.random() < 0.3
        return dict(kind="prefix", model=model, dtype=dtype, layers=2 if last else 1, lens=_texts(lens), mrope=True if last else rng.random() < 0.5,
                    last_rows=last, hidden=not last and rng.random() < 0.3)
    if kind == "suffix":
        n_prefix, group = rng.randint(1, 4), rng.choice([1, 1, 1, 4, 8])
        longest = min(_spread(rng, 16, 1024), 10000 // (n_prefix * group))
        return dict(kind="suffix", model=rng.choice(["7b", "7b", "32b"]), dtype=dtype, layers=1,
                    prefix=_texts(_spread(rng, 300, 12288) for _ in range(n_prefix)), group=group,
                    lens=_texts(rng.randint(max(1, longest // 4), longest) for _ in range(n_prefix * group)), fused=rng.random() < 0.5)
    if kind == "prompt":
        rows = _spread(rng, 16, 2048)
        return dict(kind="prompt", model="7b", dtype=dtype, layers=1, lens=_texts([rows * 2 + rng.randint(1, 2000), rows * 2 + rng.randint(1, 2000)]),
                    rows=rows, fused=rng.random() < 0.5)
    n = rng.randint(1, 4)
    return dict(kind="both", model="tiny", dtype="f32", layers=2, prefix=_texts(_spread(rng, 32, 1024) for _ in range(n)),
                lens=_texts(_spread(rng, 4, 128) for _ in range(n)))


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _shape(case) -> ModelShape:
    return replace(MODELS[case["model"]], n_layers=int(case["layers"]), dtype=case["dtype"])


def _lens(case, key="lens"):
    return [int(x) for x in str(case[key]).split(",")]


def _cu(lens):
    out = [0]
    for n in lens:
        out.append(out[-1] + n)
    return out


def _torch_dtype(m):
    return {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[m.dtype]


class _Draw:
    """Seeded draws on the GPU, one stream per tensor name."""

    def __init__(self, seed):
        self.seed = int(seed)

    def _gen(self, name):
        g = torch.Generator(device="cuda")
        g.manual_seed((self.seed * 1000003 + zlib.crc32(name.encode())) & 0x7FFFFFFFFFFF)
        return g

    def normal(self, name, shape, std, dtype, mean=0.0):
        t = torch.empty(shape, dtype=dtype, device="cuda")
        return t.normal_(mean, std, generator=self._gen(name))

    def ints(self, name, n, lo, hi):
        return torch.randint(lo, hi, (n,), dtype=torch.int32, device="cuda", generator=self._gen(name))


def _weights(m: ModelShape, d: _Draw):
    dt, e, hd = _torch_dtype(m), m.d_model, m.head_dim
    layers = []
    for l in range(m.n_layers):
        w = lambda n, *s: d.normal(f"{n}.{l}", s, 0.02, dt)
        layers.append(dict(wq=w("wq", m.n_q_heads * hd, e), wk=w("wk", m.n_kv_heads * hd, e), wv=w("wv", m.n_kv_heads * hd, e),
                           wo=w("wo", e, m.n_q_heads * hd), w_gate=w("w_gate", m.ffn_dim, e), w_up=w("w_up", m.ffn_dim, e),
                           w_down=w("w_down", e, m.ffn_dim),
                           attn_norm=d.normal(f"an.{l}", (e,), 0.1, dt, 1.0), mlp_norm=d.normal(f"mn.{l}", (e,), 0.1, dt, 1.0),
                           bq=d.normal(f"bq.{l}", (m.n_q_heads * hd,), 0.1, dt), bk=d.normal(f"bk.{l}", (m.n_kv_heads * hd,), 0.1, dt),
                           bv=d.normal(f"bv.{l}", (m.n_kv_heads * hd,), 0.1, dt)))
    return dict(embed=d.normal("embed", (m.vocab, e), 0.02, dt), lm_head=d.normal("lm_head", (m.vocab, e), 0.02, dt),
                final_norm=d.normal("final_norm", (e,), 0.1, dt, 1.0), layers=layers)


class Model(DeviceModel):
    """A DeviceModel over weights that are already on the GPU."""

    def __init__(self, m: ModelShape, weights, max_position=MAX_POSITION):
        self.shape, self.device, self.dtype, self.max_position = m, torch.device("cuda"), _torch_dtype(m), max_position
        self.embed, self.lm_head, self.final_norm, self.layers = (weights[k] for k in ("embed", "lm_head", "final_norm", "layers"))
        arr = (rb.RpLayerWeights * m.n_layers)()
        for i, lw in enumerate(self.layers):
            for name, _ in rb.RpLayerWeights._fields_:
                setattr(arr[i], name, lw[name].data_ptr())
        self._layer_arr = arr
        self._weights = rb.RpWeights(self.embed.data_ptr(), self.final_norm.data_ptr(), self.lm_head.data_ptr(), arr)
        self.config = rb.make_config(m, max_position, 0)
        self.handle = rb.rp_create(self.config, self._weights)


def _prompt_ids(m, d: _Draw, lens):
    """Packed ids, one block of visual slots (-1) and then text per prompt, and the slots' count."""
    ids = d.ints("ids", sum(lens), 0, m.vocab)
    n_vis, o = 0, 0
    for n in lens:
        v = n - max(1, int(n * TEXT_SHARE))
        ids[o:o + v] = -1
        n_vis += v
        o += n
    return ids, n_vis


def _mrope_positions(m, lens):
    """[3, T] positions: visual tokens on a (time, height, width) grid 16 wide and 16 high, text after it."""
    parts, nexts = [], []
    for n in lens:
        v = n - max(1, int(n * TEXT_SHARE))
        i = torch.arange(v, dtype=torch.int32, device="cuda")
        grid = torch.stack([2 * (i // 256), i // 16 % 16, i % 16])
        first = int(max(2 * ((v - 1) // 256), 15)) + 1
        text = torch.arange(first, first + n - v, dtype=torch.int32, device="cuda").expand(3, -1)
        parts.append(torch.cat([grid, text], 1))
        nexts.append(first + n - v)
    return torch.cat(parts, 1).contiguous(), nexts


def _sections(m):
    half = m.head_dim // 2
    return [half // 4, half * 3 // 8, half * 3 // 8]


def _kv_spread(m):
    return 0.02 * math.sqrt(m.d_model)


def _inputs(case, seed):
    """Everything a call takes beside its outputs and scratch."""
    m, d, kind = _shape(case), _Draw(seed), case["kind"]
    dt, s = _torch_dtype(m), {}
    s["weights"] = _weights(m, d)
    if kind in ("prefix", "both"):
        lens = _lens(case, "lens" if kind == "prefix" else "prefix")
        s["cu"] = _cu(lens)
        s["ids"], n_vis = _prompt_ids(m, d, lens)
        s["visual"] = d.normal("visual", (n_vis, m.d_model), 1.0, dt)
        if case.get("mrope"):
            s["positions"], _ = _mrope_positions(m, lens)
    if kind in ("suffix", "both"):
        plens, slens = _lens(case, "prefix"), _lens(case)
        s["prefix_cu"], s["suffix_cu"] = _cu(plens), _cu(slens)
        s["response"] = d.ints("response", sum(slens), 0, m.vocab)
        s["group"] = int(case.get("group", 1))
    if kind == "suffix":
        shape = (m.n_layers, sum(plens), m.n_kv_heads, m.head_dim)
        s["K"], s["V"] = d.normal("K", shape, _kv_spread(m), dt), d.normal("V", shape, _kv_spread(m), dt)
        s["h_last"] = d.normal("h_last", (len(plens), m.d_model), 1.5, torch.float32)
    if kind == "prompt":
        lens, rows = _lens(case), int(case["rows"])
        s["cu"] = _cu(lens)
        s["ids"] = d.ints("ids", sum(lens), 0, m.vocab)
        s["hidden"] = d.normal("hidden", (sum(lens), m.d_model), 1.5, torch.float32)
        # the text at each prompt's end
        per = [rows // len(lens) + (1 if i < rows % len(lens) else 0) for i in range(len(lens))]
        s["rows"] = torch.cat([torch.arange(s["cu"][i + 1] - n, s["cu"][i + 1], dtype=torch.int32, device="cuda") for i, n in enumerate(per)])
    if kind == "decode":
        B, cap = int(case["batch"]), int(case["kv_hi"]) + 64
        shape = (m.n_layers, B, cap, m.n_kv_heads, m.head_dim)
        s["K"], s["V"] = d.normal("K", shape, _kv_spread(m), dt), d.normal("V", shape, _kv_spread(m), dt)
        s["kv_len"] = d.ints("kv_len", B, int(case["kv_lo"]), int(case["kv_hi"]) + 1)
        s["ids"] = d.ints("ids", B, 0, m.vocab)
    return m, s


def prepare(case, seed):
    m, s = _inputs(case, seed)
    kind = s["kind"] = case["kind"]
    s["model"] = model = Model(m, s.pop("weights"))
    if kind in ("prefix", "both"):
        B, T = len(s["cu"]) - 1, s["cu"][-1]
        s["kv"] = model.alloc_kv(T)
        s["h"] = torch.empty((B, m.d_model), dtype=torch.float32, device="cuda")
        if case.get("hidden"):
            s["hidden"] = torch.empty((T, m.d_model), dtype=torch.float32, device="cuda")
        s["flags"] = rb.RP_PREFIX_LAST_ROWS_ONLY if case.get("last_rows") else 0
        s["ws"] = model.workspace(rb.rp_prefix_workspace_bytes(model.handle, B, s["cu"]))
    if kind in ("suffix", "both"):
        flags = rb.RP_SUFFIX_FUSED_LOGPROB if case.get("fused") else 0
        s["fused"] = flags
        s["lp"] = torch.empty(s["suffix_cu"][-1], dtype=torch.float32, device="cuda")
        P, S = len(s["prefix_cu"]) - 1, len(s["suffix_cu"]) - 1
        s["of"] = [i // s["group"] for i in range(S)]
        if s["group"] > 1 or flags:
            n = rb.rp_suffix_grouped_workspace_bytes(model.handle, P, s["prefix_cu"], S, s["of"], s["suffix_cu"], flags)
        else:
            n = rb.rp_suffix_workspace_bytes(model.handle, P, s["prefix_cu"], s["suffix_cu"])
        s["ws2"] = model.workspace(n)
    if kind == "prompt":
        s["fused"] = rb.RP_SUFFIX_FUSED_LOGPROB if case["fused"] else 0
        s["lp"] = torch.empty(s["rows"].numel(), dtype=torch.float32, device="cuda")
        s["ws"] = model.workspace(rb.rp_prompt_logprob_workspace_bytes(model.handle, s["rows"].numel(), s["fused"]))
    if kind == "decode":
        B, cap = s["K"].shape[1], s["K"].shape[2]
        s["logits"] = torch.empty((B, m.vocab), dtype=torch.float32, device="cuda")
        s["next"] = torch.empty(B, dtype=torch.int32, device="cuda")
        s["ws"] = model.workspace(rb.rp_decode_workspace_bytes(model.handle, B, cap))
    return s


def _run_prefix(s):
    model, positions = s["model"], s.get("positions")
    K, V, h = model.prefix(s["cu"], s["ids"], s["visual"], kv=s["kv"], h_last=s["h"], hidden_out=s.get("hidden"), workspace=s["ws"], positions=positions,
                           mrope_section=_sections(model.shape) if positions is not None else None, flags=s["flags"])
    return dict(K=K, V=V, h_last=h, hidden=s.get("hidden"))


def _run_suffix(s, K, V, h):
    model = s["model"]
    if s["group"] > 1 or s["fused"]:
        return model.suffix_grouped(s["prefix_cu"], s["of"], s["suffix_cu"], K, V, h, s["response"], logprobs=s["lp"],
                                    workspace=s["ws2"], flags=s["fused"])
    return model.suffix(s["prefix_cu"], s["suffix_cu"], K, V, h, s["response"], logprobs=s["lp"], workspace=s["ws2"])


def run(s):
    kind, model = s["kind"], s["model"]
    if kind == "prefix":
        return _run_prefix(s)
    if kind == "suffix":
        return dict(logprobs=_run_suffix(s, s["K"], s["V"], s["h_last"]))
    if kind == "prompt":
        return dict(logprobs=model.prompt_logprobs(s["cu"], s["ids"], s["hidden"], s["rows"], logprobs=s["lp"], workspace=s["ws"], flags=s["fused"]))
    if kind == "decode":
        ids = model.decode(s["K"], s["V"], s["kv_len"], s["ids"], logits=s["logits"], next_ids=s["next"], workspace=s["ws"])
        return dict(logits=s["logits"], next_ids=ids, K=s["K"], V=s["V"])  # the cache holds the new row
    out = _run_prefix(s)
    out["logprobs"] = _run_suffix(s, out["K"], out["V"], out["h_last"])
    return out


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def work(case):
    m, kind = _shape(case), case["kind"]
    es = 4 if m.dtype == "f32" else 2
    hq, kvd = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    layer, head = m.params_per_layer, m.vocab * m.d_model
    by = fl = 0.0

    def prefix(lens, last_rows):
        T, L, B = sum(lens), m.n_layers, len(lens)
        b = L * layer * es + T * m.d_model * es + L * T * 2 * kvd * es + B * m.d_model * 4 + (T * m.d_model * 4 if case.get("hidden") else 0)
        full = L - 1 if last_rows else L
        f = full * (2.0 * T * layer + sum(2.0 * hq * n * (n + 1) for n in lens))
        if last_rows:
            f += 2.0 * T * m.d_model * 2 * kvd + 2.0 * B * (layer - m.d_model * 2 * kvd) + sum(4.0 * hq * n for n in lens)
        return b, f

    def suffix(plens, slens, group):
        R, L = sum(slens), m.n_layers
        b = L * layer * es + head * es + R * m.d_model * es + L * sum(plens) * 2 * kvd * es + len(plens) * m.d_model * 4 + R * 8
        f = 2.0 * R * (L * layer + head)
        for i, n in enumerate(slens):
            f += L * 4.0 * hq * (n * plens[i // group] + n * (n + 1) / 2)
        return b, f

    if kind in ("prefix", "both"):
        by, fl = prefix(_lens(case, "lens" if kind == "prefix" else "prefix"), bool(case.get("last_rows")))
    if kind in ("suffix", "both"):
        b, f = suffix(_lens(case, "prefix"), _lens(case), int(case.get("group", 1)))
        by, fl = by + b, fl + f
    if kind == "prompt":
        n = int(case["rows"])
        by, fl = head * es + n * m.d_model * 4 + n * 12, 2.0 * n * head
    if kind == "decode":
        B, keys = int(case["batch"]), int(case["batch"]) * (int(case["kv_lo"]) + int(case["kv_hi"])) / 2 + int(case["batch"])
        by = m.n_layers * layer * es + head * es + m.n_layers * keys * 2 * kvd * es + B * (m.d_model * es + m.vocab * 4 + 12)
        fl = 2.0 * B * (m.n_layers * layer + head) + m.n_layers * 4.0 * hq * keys
    return dict(bytes=by, flops=fl)


# About four times the relative error against 64-bit arithmetic (worst case seen: bf16 K/V 0.0037,
# h_last and hidden 0.0099, decode logits 0.012, log-probs 0.001; fp16 an eighth of that: 3 more
# bits; fp32 6e-7).  The largest single difference follows the spread of the many small ones.
def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    k = 1.0 if case["dtype"] == "bf16" else 0.15
    if case["kind"] in ("suffix", "prompt"):
        return {"rel": 4e-3 * k, "max": 2e-2 * k}
    if case["kind"] == "decode":
        return {"rel": 3e-2 * k, "max": 0.3 * k, "differ": 0.01}
    return {"rel": 3e-2 * k, "max": 0.25 * k}


# ------------------------------------------------------------------------------------------
# the same in 64 bits, with torch alone
# ------------------------------------------------------------------------------------------
def _norm(x, w, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * w


def _rotate(x, cos, sin):
    """x [n, heads, D] by cos, sin [n, D/2] (rotate-half pairs)."""
    h = x.shape[-1] // 2
    a, b, c, s = x[..., :h], x[..., h:], cos[:, None], sin[:, None]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _angles(m, pos):
    """cos, sin [n, D/2] of positions [n] or [3, n] (multimodal sections)."""
    half = m.head_dim // 2
    inv = m.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / m.head_dim)
    if pos.dim() == 2:
        sec = torch.tensor(sum(([k] * n for k, n in enumerate(_sections(m))), []), device="cuda")
        t = pos.double()[sec].T * inv
    else:
        t = pos.double()[:, None] * inv
    return torch.cos(t), torch.sin(t)


def _attend(m, q, k, v, first):
    """q [n, Hq, D] at key indices first .. over k, v [keys, Hkv, D] -> [n, Hq D]."""
    n, G = q.shape[0], m.group
    out = torch.empty_like(q)
    for g in range(m.n_kv_heads):
        kg, vg = k[:, g].T.contiguous(), v[:, g].contiguous()
        for h in range(g * G, g * G + G):
            for i in range(0, n, 2048):
                e = min(n, i + 2048)
                keys = first + e
                s = (q[i:e, h].contiguous() @ kg[:, :keys].contiguous()) / math.sqrt(m.head_dim)
                mask = torch.arange(keys, device="cuda")[None] > (first + torch.arange(i, e, device="cuda"))[:, None]
                s.masked_fill_(mask, -math.inf)
                out[i:e, h] = torch.softmax(s, -1) @ vg[:keys]
    return out.reshape(n, -1)


def _layer(m, w, x, cos, sin, attend):
    """One decoder layer over rows x; attend(q, k, v) gives the attention rows."""
    n, D = x.shape[0], m.head_dim
    f = lambda t: t.double()
    h = _norm(x, f(w["attn_norm"]), m.rms_eps)
    q = (h @ f(w["wq"]).T + f(w["bq"])).reshape(n, m.n_q_heads, D)
    k = (h @ f(w["wk"]).T + f(w["bk"])).reshape(n, m.n_kv_heads, D)
    v = (h @ f(w["wv"]).T + f(w["bv"])).reshape(n, m.n_kv_heads, D)
    q, k = _rotate(q, cos, sin), _rotate(k, cos, sin)
    x = x + attend(q, k, v) @ f(w["wo"]).T
    h = _norm(x, f(w["mlp_norm"]), m.rms_eps)
    wg, wu, wd = f(w["w_gate"]), f(w["w_up"]), f(w["w_down"])
    y = torch.empty_like(x)
    for i in range(0, n, 4096):
        g = h[i:i + 4096] @ wg.T
        y[i:i + 4096] = (g * torch.sigmoid(g) * (h[i:i + 4096] @ wu.T)) @ wd.T
    return x + y, k, v


def _exact_prefix(m, s):
    w, cu = s["weights"], s["cu"]
    ids = s["ids"].long()
    vis = ids < 0
    x = w["embed"][ids.clamp(min=0)].double()
    x[vis] = s["visual"].double()[: int(vis.sum())]
    pos = s.get("positions")
    if pos is None:
        pos = torch.cat([torch.arange(cu[b + 1] - cu[b], device="cuda") for b in range(len(cu) - 1)])
    cos, sin = _angles(m, pos)

    def attend(q, k, v):
        return torch.cat([_attend(m, q[a:b], k[a:b], v[a:b], 0) for a, b in zip(cu[:-1], cu[1:])])

    Ks, Vs = [], []
    for lw in w["layers"]:
        x, k, v = _layer(m, lw, x, cos, sin, attend)
        Ks.append(k)
        Vs.append(v)
    last = torch.tensor([c - 1 for c in cu[1:]], device="cuda")
    return dict(K=torch.stack(Ks), V=torch.stack(Vs), h_last=x[last], hidden=x if s.get("keep_hidden") else None)


def _score(m, w, rows, ids):
    """log p(ids) from final hidden rows."""
    h, out = _norm(rows, w["final_norm"].double(), m.rms_eps), []
    lm = w["lm_head"].double()
    for i in range(0, h.shape[0], 512):
        z = h[i:i + 512] @ lm.T
        out.append(z.gather(1, ids[i:i + 512, None].long())[:, 0] - torch.logsumexp(z, 1))
    return torch.cat(out)


def _exact_suffix(m, s, K, V, h_last):
    w, pcu, scu, group = s["weights"], s["prefix_cu"], s["suffix_cu"], s["group"]
    S = len(scu) - 1
    x = w["embed"][s["response"].long()].double()
    plen = [pcu[p + 1] - pcu[p] for p in range(len(pcu) - 1)]
    pos = torch.cat([plen[i // group] + torch.arange(scu[i + 1] - scu[i], device="cuda") for i in range(S)])
    cos, sin = _angles(m, pos)
    for l, lw in enumerate(w["layers"]):
        def attend(q, k, v):
            parts = []
            for i in range(S):
                p, a, b = i // group, scu[i], scu[i + 1]
                kk = torch.cat([K[l, pcu[p]:pcu[p + 1]].double(), k[a:b]])
                vv = torch.cat([V[l, pcu[p]:pcu[p + 1]].double(), v[a:b]])
                parts.append(_attend(m, q[a:b], kk, vv, plen[p]))
            return torch.cat(parts)

        x, _, _ = _layer(m, lw, x, cos, sin, attend)
    prev = torch.cat([x.new_zeros(1, x.shape[1]), x[:-1]])
    for i in range(S):
        prev[scu[i]] = h_last[i // group].double()
    return _score(m, w, prev, s["response"])


def exact(case, seed):
    m, s = _inputs(case, seed)
    kind, w = case["kind"], s["weights"]
    if kind == "prefix":
        s["keep_hidden"] = bool(case.get("hidden"))
        return _exact_prefix(m, s)
    if kind == "suffix":
        return dict(logprobs=_exact_suffix(m, s, s["K"], s["V"], s["h_last"]))
    if kind == "both":
        out = _exact_prefix(m, s)
        out["logprobs"] = _exact_suffix(m, s, out["K"], out["V"], out["h_last"])
        return out
    if kind == "prompt":
        t = s["rows"].long()
        return dict(logprobs=_score(m, w, s["hidden"][t - 1].double(), s["ids"][t]))
    n = s["kv_len"].long()
    x = w["embed"][s["ids"].long()].double()
    cos, sin = _angles(m, n)
    for l, lw in enumerate(w["layers"]):
        def attend(q, k, v):
            parts = []
            for b, nb in enumerate(n.tolist()):
                kk = torch.cat([s["K"][l, b, :nb].double(), k[b:b + 1]]).permute(1, 2, 0).contiguous()  # [Hkv, D, keys]
                vv = torch.cat([s["V"][l, b, :nb].double(), v[b:b + 1]]).permute(1, 0, 2).contiguous()
                a = torch.softmax(torch.bmm(q[b].reshape(m.n_kv_heads, m.group, -1), kk) / math.sqrt(m.head_dim), -1)
                parts.append(torch.bmm(a, vv).reshape(1, -1))
            return torch.cat(parts)

        x, _, _ = _layer(m, lw, x, cos, sin, attend)
    logits = _norm(x, w["final_norm"].double(), m.rms_eps) @ w["lm_head"].double().T
    return dict(logits=logits, next_ids=None, K=None, V=None)
