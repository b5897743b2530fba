"""Measured cases: what a program that decodes speculatively with this library has it do.

Four kinds of call, each through the public entry points of paper_2404_08856_amd.spd:

  accept   accept / resample of drafted tokens (spd_speculative_accept)
  draft    the draft's part of a block: gamma sequential draft steps, D rows and tokens written in place
  prefill  the prompt into the KV cache (spd_prefill / spd_prefill_tokens), with the keys and values it leaves
  verify   two consecutive target calls per sequence with the rollback of the rejected positions between them

Shapes: the LLaMA-7B layer shape (four layers and the LM head, or all 32 layers), the 12-layer 110M draft and
the paper's 4-layer draft.  Sizes: 1 to 64 sequences in the accept step, 1 to 8 in the models, 1 to 8 tokens
per sequence and call, contexts of 64 to 2048 positions.
"""
import math

import torch

from paper_2404_08856_amd import spd, synth

DEV = "cuda"


def listed():
    return [
        # one conversation: the accept step of one block as the block loop calls it (target logits, draft
        # probabilities).  The smallest call there is: launches and dependent round trips.
        {"name": "accept_1x4", "kind": "accept", "n_seqs": 1, "gamma": 4, "vocab": 32000, "draft_probs": True, "temperature": 1.0},
        # a full serving batch, both sides logits: the largest accept step
        {"name": "accept_64x4", "kind": "accept", "n_seqs": 64, "gamma": 4, "vocab": 32000, "draft_probs": False, "temperature": 1.0},
        # one conversation: the draft steps of one block after a short prompt (deep narrow draft: chains of small launches)
        {"name": "draft_110m_1x4", "kind": "draft", "shape": "draft_110m", "layers": 12, "n_seqs": 1, "gamma": 4, "context": 66, "temperature": 1.0},
        # eight conversations on the paper's own draft shape, 1472 text positions each, draft length 5
        {"name": "draft_115m_8x5", "kind": "draft", "shape": "draft_paper_115m", "layers": 4, "n_seqs": 8, "gamma": 5, "context": 1472, "temperature": 1.0},
        # the text-only draft takes in a long prompt
        {"name": "prefill_draft_1472", "kind": "prefill", "shape": "draft_110m", "layers": 12, "rows": 1472, "image_rows": 0},
        # the target takes in one image and a short question
        {"name": "prefill_640", "kind": "prefill", "shape": "llama7b", "layers": 4, "rows": 640, "image_rows": 576},
        # the target takes in one image and a long text, ragged length
        {"name": "prefill_2047", "kind": "prefill", "shape": "llama7b", "layers": 4, "rows": 2047, "image_rows": 576},
        # one conversation, draft length 5: more rows than one operand tile holds
        {"name": "verify_1x6", "kind": "verify", "shape": "llama7b", "layers": 4, "n_seqs": 1, "tokens": 6, "context": 640},
        # eight conversations decoded without a draft (the baseline speculative decoding is compared with)
        {"name": "verify_8x1", "kind": "verify", "shape": "llama7b", "layers": 4, "n_seqs": 8, "tokens": 1, "context": 2048},
        # three conversations, draft length 4: a small batch
        {"name": "verify_3x5", "kind": "verify", "shape": "llama7b", "layers": 4, "n_seqs": 3, "tokens": 5, "context": 700},
        # eight conversations, draft length 4, long contexts: the serving batch
        {"name": "verify_8x5", "kind": "verify", "shape": "llama7b", "layers": 4, "n_seqs": 8, "tokens": 5, "context": 2048},
        # the whole 7B model, one conversation, draft length 4: the call everything else serves
        {"name": "verify_7b_1x5", "kind": "verify", "shape": "llama7b", "layers": 32, "n_seqs": 1, "tokens": 5, "context": 640},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["accept", "draft", "prefill", "verify", "verify"])
    if kind == "accept":
        vocab = rng.choice([32000, _log_int(rng, 1000, 40000), 16 * _log_int(rng, 64, 2500)])
        return {"kind": kind, "n_seqs": _log_int(rng, 1, 64), "gamma": rng.randint(1, 7), "vocab": vocab,
                "draft_probs": rng.random() < 0.5, "temperature": rng.choice([0.0, 0.7, 1.0])}
    if kind == "draft":
        shape = rng.choice(["draft_110m", "draft_paper_115m"])
        return {"kind": kind, "shape": shape, "layers": synth.SHAPES[shape].n_layers, "n_seqs": rng.randint(1, 8), "gamma": rng.randint(1, 7),
                "context": _log_int(rng, 64, 2000), "temperature": rng.choice([0.7, 1.0])}
    if kind == "prefill":
        shape = rng.choice(["draft_110m", "draft_paper_115m", "llama7b", "llama7b"])
        rows = _log_int(rng, 16, 2047 if shape == "llama7b" else 1472)
        layers = 4 if shape == "llama7b" else synth.SHAPES[shape].n_layers
        return {"kind": kind, "shape": shape, "layers": layers, "rows": rows, "image_rows": min(576, rows // 2) if shape == "llama7b" else 0}
    return {"kind": kind, "shape": "llama7b", "layers": 4, "n_seqs": rng.randint(1, 8), "tokens": rng.randint(1, 8), "context": _log_int(rng, 64, 2048)}


# ---- inputs ---------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _shape(case):
    s = synth.SHAPES[case["shape"]]
    return s if s.n_layers == case["layers"] else synth.llama7b_layers(case["layers"])


def _weights(case, seed, g):
    """N(0, 0.02) matrices, norm gains around 1."""
    shape = _shape(case)
    w = synth.make_weights(shape, seed, device=DEV)
    gain = lambda: 1.0 + 0.1 * torch.randn(shape.d_model, generator=g, device=DEV)
    w["final_norm"] = gain()
    for lw in w["layers"]:
        lw["attn_norm"], lw["mlp_norm"] = gain(), gain()
    return w


def _tokens(shape, vocab, g):
    return torch.randint(0, vocab, shape, generator=g, device=DEV, dtype=torch.int32)


def _uniforms(shape, g):
    return torch.randint(0, 1 << 24, shape, generator=g, device=DEV).float() * 2.0 ** -24


def _contexts(case):
    """Cached positions of each sequence before the call: the longest first, the others a little shorter."""
    return [max(2, case["context"] - (37 * s) % max(1, case["context"] // 2)) for s in range(case["n_seqs"])]


def _prompt(case, rows, w, g):
    """float32 input rows of one sequence: image rows ~ N(0, 1), then text embeddings."""
    image = case.get("image_rows", min(576, rows // 2))
    text = _tokens((rows - image,), w["embed"].shape[0], g)
    return torch.cat([torch.randn((image, w["embed"].shape[1]), generator=g, device=DEV), w["embed"][text.long()].float()]).contiguous()


def _accept_inputs(case, seed):
    g = _gen(seed)
    n, gamma, V = case["n_seqs"], case["gamma"], case["vocab"]
    target = 2.0 * torch.randn((n, gamma + 1, V), generator=g, device=DEV)
    draft = target[:, :gamma] + torch.randn((n, gamma, V), generator=g, device=DEV)
    temp = case["temperature"] if case["temperature"] > 0 else 1.0
    probs = torch.softmax(draft.double() / temp, -1)
    tokens = torch.multinomial(probs.reshape(-1, V).float(), 1, generator=g).reshape(n, gamma).to(torch.int32)
    if case["temperature"] == 0:
        tokens = draft.argmax(-1).to(torch.int32)
        probs = torch.nn.functional.one_hot(draft.argmax(-1), V)
    return {"target": target, "draft": probs.float().contiguous() if case["draft_probs"] else draft.contiguous(),
            "tokens": tokens.contiguous(), "u": _uniforms((n, gamma + 1), g)}


def _model_inputs(case, seed):
    """Everything but the model itself, from the seed alone."""
    g = _gen(seed)
    w = _weights(case, seed, g)
    V = _shape(case).vocab
    s = {"weights": w}
    if case["kind"] == "prefill":
        if case["image_rows"]:
            s["rows"] = _prompt(case, case["rows"], w, g)
        else:
            s["ids"] = _tokens((case["rows"],), V, g)
    elif case["kind"] == "draft":
        n, gamma = case["n_seqs"], case["gamma"]
        s["contexts"] = _contexts(case)
        s["prompts"] = [_tokens((c,), V, g) for c in s["contexts"]]
        # The tokens each step takes in are given, so that one draw that falls on another side of a rounding
        # does not make every later step a different computation.
        s["inputs"] = _tokens((n, gamma + 1), V, g)
        s["u"] = _uniforms((n, gamma), g)
    else:
        n, M = case["n_seqs"], case["tokens"]
        s["contexts"] = _contexts(case)
        s["prompts"] = [_prompt(case, c, w, g) for c in s["contexts"]]
        s["blocks"] = [_tokens((n, M), V, g) for _ in range(2)]
        # positions that stay of the first block (accepted tokens and the one before them)
        s["kept"] = (torch.randint(0, M, (n,), generator=g, device=DEV) + 1).tolist()
    return s


def prepare(case, seed):
    """Inputs, model and buffers a program holds before the call; the prompts are already in the KV cache."""
    if case["kind"] == "accept":
        s = _accept_inputs(case, seed)
        n, gamma = case["n_seqs"], case["gamma"]
        s.update(case=case, out=torch.zeros((2, n), dtype=torch.int32, device=DEV), prob=torch.zeros((n, gamma), device=DEV),
                 workspace=torch.empty(spd.spd_accept_workspace_bytes(n, gamma, case["vocab"]), dtype=torch.uint8, device=DEV))
        return s
    s = _model_inputs(case, seed)
    shape = _shape(case)
    kind = case["kind"]
    n = case.get("n_seqs", 1)
    positions = case["rows"] if kind == "prefill" else case["context"] + (case["gamma"] + 1 if kind == "draft" else 2 * case["tokens"])
    model = spd.Model(spd.make_config(shape, n, positions), s.pop("weights"))
    s.update(case=case, model=model)
    V = shape.vocab
    if kind == "prefill":
        s["logits"] = torch.zeros(V, device=DEV)
        s["k"], s["v"] = (torch.zeros((shape.n_layers, case["rows"], shape.n_heads, shape.head_dim), device=DEV) for _ in range(2))
        return s
    for i, p in enumerate(s.pop("prompts")):
        (model.spd_prefill_tokens if kind == "draft" else model.spd_prefill)(i, p)
    if kind == "draft":
        s["D"] = torch.zeros((n, case["gamma"], V), device=DEV)
        s["drawn"] = torch.zeros((n, case["gamma"]), dtype=torch.int32, device=DEV)
    else:
        s["out"] = [torch.zeros((n, case["tokens"], V), device=DEV) for _ in range(2)]
    return s


# ---- one pass -------------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "accept":
        spd.spd_speculative_accept(s["target"], s["draft"], s["tokens"], s["u"], case["temperature"],
                                   spd.SPD_DRAFT_IS_PROBS if case["draft_probs"] else 0, s["out"][0], s["out"][1], s["prob"], s["workspace"])
        return {"accepted_and_next": s["out"], "prob": s["prob"]}
    m = s["model"]
    if kind == "prefill":
        m.spd_kv_set_len([0])
        if "rows" in s:
            m.spd_prefill(0, s["rows"], s["logits"])
        else:
            m.spd_prefill_tokens(0, s["ids"], s["logits"])
        for l in range(case["layers"]):
            m.spd_kv_export(l, 0, 0, s["k"][l], s["v"][l])
        return {"logits": s["logits"], "k": s["k"], "v": s["v"]}
    if kind == "draft":
        n, gamma = case["n_seqs"], case["gamma"]
        D, drawn, V = s["D"], s["drawn"], s["D"].shape[2]
        m.spd_kv_set_len(s["contexts"])
        for j in range(gamma):                  # the first step takes two tokens: a block starts one position back
            m.spd_draft_step_strided(s["inputs"][:, 0 if j == 0 else j + 1:], gamma + 1, n, 2 if j == 0 else 1, case["temperature"], s["u"][:, j:], gamma,
                                     D[:, j:], gamma * V, drawn[:, j:], gamma)
        return {"D": D, "drawn": drawn}
    m.spd_kv_set_len(s["contexts"])
    m.spd_verify_forward(s["blocks"][0], s["out"][0])
    m.spd_kv_set_len([c + k for c, k in zip(s["contexts"], s["kept"])])
    m.spd_verify_forward(s["blocks"][1], s["out"][1])
    return {"first": s["out"][0], "second": s["out"][1]}


# ---- what a pass cannot do without ----------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "accept":
        rows = case["n_seqs"] * (2 * case["gamma"] + 1)
        return {"bytes": 4 * rows * case["vocab"], "flops": 4 * rows * case["vocab"]}
    shape = _shape(case)
    HD = shape.n_heads * shape.head_dim
    head = shape.vocab * shape.d_model
    layers = shape.streamed_weight_bytes() // 2 - head
    kv = 4 * HD * shape.n_layers                          # bytes of K and V of one position
    att = 4 * HD * shape.n_layers                         # operations of one (query, key) pair, all layers
    if kind == "prefill":
        n = case["rows"]
        return {"bytes": 2 * (layers + head) + n * (4 * shape.d_model + kv) + n * 2 * kv + n * kv, "flops": 2 * (layers * n + head) + att * n * n // 2}
    ctx = _contexts(case)
    if kind == "draft":
        calls, rows = case["gamma"], case["n_seqs"] * (case["gamma"] + 1)
        out = 4 * case["n_seqs"] * case["gamma"] * shape.vocab
        return {"bytes": calls * (2 * (layers + head) + kv * sum(ctx)) + out, "flops": 2 * (layers + head) * rows + att * rows * max(ctx)}
    rows = 2 * case["n_seqs"] * case["tokens"]
    return {"bytes": 4 * (layers + head) + 2 * kv * sum(ctx) + kv * rows + 4 * rows * shape.vocab,
            "flops": 2 * (layers + head) * rows + att * rows * sum(ctx) // len(ctx)}


def tolerance(case):
    """Largest difference another correct implementation at this precision shows.

    Accept: float32 softmax, a few 1e-7 per probability; a draw moves to a neighbouring token where the threshold
    sits within that of a boundary.  Models: float32 arithmetic on bf16 weights, but K and V are rounded to bf16,
    which turns a last-bit difference into a flipped rounding now and then; it grows with the depth.  Measured
    against exact(): draft rows up to 9e-5, logits 2e-4 to 4.4e-4 and K, V 5.7e-4 at four layers, 1.1e-3 at 32 layers.
    """
    if case["kind"] == "accept":
        return {"rel": 1e-5, "differ": 0.5 if case["n_seqs"] < 8 else 0.05}
    if case["kind"] == "draft":
        return {"rel": 4e-4, "differ": 0.5 if case["n_seqs"] * case["gamma"] < 20 else 0.15}
    return {"rel": 5e-3 if case["layers"] > 12 else 2e-3}


# ---- the same in 64 bits --------------------------------------------------------------------------

class _Decoder:
    """LLaMA decoder in float64 with a bf16-rounded KV cache, one sequence."""

    def __init__(self, shape, w):
        self.c, self.w = shape, w
        self.k = [None] * shape.n_layers
        self.v = [None] * shape.n_layers
        self.kept = 0

    def _norm(self, x, gain):
        return x / torch.sqrt(x.square().mean(-1, keepdim=True) + self.c.rms_eps) * gain.double()

    def _rope(self, x, pos):
        half = self.c.head_dim // 2
        freq = self.c.rope_theta ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / self.c.head_dim)
        ang = pos.double()[:, None] * freq
        cos, sin = ang.cos()[:, None], ang.sin()[:, None]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def _attend(self, q, k, v, pos):
        out = torch.empty_like(q)
        keys = torch.arange(k.shape[0], device=DEV)
        for h in range(self.c.n_heads):
            sc = q[:, h] @ k[:, h].T / math.sqrt(self.c.head_dim)
            sc = sc.masked_fill(keys[None] > pos[:, None], -math.inf)
            out[:, h] = torch.softmax(sc, -1) @ v[:, h]
        return out.reshape(q.shape[0], -1)

    def forward(self, x, n_logits):
        """x float64 [n, d]; appends n positions, returns the logits of the last n_logits rows."""
        c = self.c
        x = x.double()
        n, pos = x.shape[0], self.kept + torch.arange(x.shape[0], device=DEV)
        for l, lw in enumerate(self.w["layers"]):
            a = self._norm(x, lw["attn_norm"])
            q, k, v = ((a @ lw[t].double().T).reshape(n, c.n_heads, c.head_dim) for t in ("wq", "wk", "wv"))
            q, k, v = self._rope(q, pos), self._rope(k, pos).to(torch.bfloat16).double(), v.to(torch.bfloat16).double()
            if self.kept:
                k, v = torch.cat([self.k[l][:self.kept], k]), torch.cat([self.v[l][:self.kept], v])
            self.k[l], self.v[l] = k, v
            x = x + self._attend(q, k, v, pos) @ lw["wo"].double().T
            b = self._norm(x, lw["mlp_norm"])
            x = x + (torch.nn.functional.silu(b @ lw["w_gate"].double().T) * (b @ lw["w_up"].double().T)) @ lw["w_down"].double().T
        self.kept += n
        head = self.w["embed"] if self.w["lm_head"] is None else self.w["lm_head"]
        return self._norm(x[n - n_logits:], self.w["final_norm"]) @ head.double().T if n_logits else None

    def embed(self, ids):
        return self.w["embed"][ids.long()].double()


def exact(case, seed):
    if case["kind"] == "accept":
        s = _accept_inputs(case, seed)
        if case["temperature"] == 0:
            return None
        T = torch.softmax(s["target"].double() / case["temperature"], -1)[:, :-1]
        D = s["draft"].double() if case["draft_probs"] else torch.softmax(s["draft"].double() / case["temperature"], -1)
        at = lambda p: p.gather(-1, s["tokens"].long()[..., None])[..., 0]
        return {"accepted_and_next": None, "prob": (at(T) / at(D)).clamp(max=1.0)}
    s = _model_inputs(case, seed)
    shape, w = _shape(case), s["weights"]
    if case["kind"] == "prefill":
        m = _Decoder(shape, w)
        logits = m.forward(s["rows"] if "rows" in s else m.embed(s["ids"]), 1)[0]
        return {"logits": logits, "k": torch.stack(m.k), "v": torch.stack(m.v)}
    if case["kind"] == "draft":
        rows = []
        for i in range(case["n_seqs"]):
            m = _Decoder(shape, w)
            m.forward(m.embed(s["prompts"][i]), 0)
            logits = m.forward(m.embed(s["inputs"][i]), case["gamma"])
            rows.append(torch.softmax(logits / case["temperature"], -1))
        return {"D": torch.stack(rows), "drawn": None}
    out = [[], []]
    for i in range(case["n_seqs"]):
        m = _Decoder(shape, w)
        m.forward(s["prompts"][i], 0)
        out[0].append(m.forward(m.embed(s["blocks"][0][i]), case["tokens"]))
        m.kept = s["contexts"][i] + s["kept"][i]
        out[1].append(m.forward(m.embed(s["blocks"][1][i]), case["tokens"]))
    return {"first": torch.stack(out[0]), "second": torch.stack(out[1])}
