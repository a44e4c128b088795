"""Workloads whose time on the GPU is measured, from a single fp32 block to
decoding steps of a large batch.

Each case goes through the entry points a program calls (``driver.Engine`` for
decoding steps, ``binding`` for the C ABI) and returns everything the call
computes.  Five kinds:

* ``decode``: two consecutive decoding steps of a batch (a full step, then a
  cache-aware one with its refresh selection on the device);
* ``block``: a call of cache-aware layers on ragged active lists, optionally
  with the attention-mass scores and the refresh selection;
* ``encode``: encoder input, encoder layers over the known tokens and the
  decoder input built from them;
* ``sample``: the diffusion sampler of the generating tokens;
* ``attend``: attention over an active and a cached key/value segment.

Inputs are drawn on the GPU from the seed.  ``exact`` recomputes a case in
float64 with plain torch operations.
"""
import math

import torch

from paper_2506_12035_amd import binding, driver, workload

DEV = "cuda"

# Decoder families (Table 1's model scales): width, heads, head width, MLP width.
FAMILIES = {"mar-b": (768, 12, 64, 3072), "mar-l": (1024, 16, 64, 4096),
            "mar-h": (1280, 16, 80, 5120)}
SEL = 2          # selection layer (1-based) of the decoding schedule
N_STEPS = 64     # decoding steps of the mask schedule
EPS = 1e-6


def listed():
    return [
        # The paper's headline batch as a service decodes it: 128 images in two
        # image ranges on two streams (8 of MAR-L's 32 layers: the time of a
        # step is proportional to the layers).
        dict(name="decode-mar-l-128", kind="decode", family="mar-l", layers=8, batch=128, n_img=256,
             n_buf=64, ratio_bp=1000, ranges=2),
        # A few images at a time: an interactive service on the small model.
        dict(name="decode-mar-b-4", kind="decode", family="mar-b", layers=12, batch=4, n_img=256,
             n_buf=64, ratio_bp=1000, ranges=1),
        # Heads of width 80 and the larger refresh ratio of the ratio sweep.
        dict(name="decode-mar-h-32", kind="decode", family="mar-h", layers=4, batch=32, n_img=256,
             n_buf=64, ratio_bp=2500, ranges=1),
        # 32x32 image tokens: long key/value sequences.
        dict(name="decode-hires-8", kind="decode", family="mar-l", layers=4, batch=8, n_img=1024,
             n_buf=64, ratio_bp=1000, ranges=2),
        # The single-block fp32 configuration: the smallest call, 32 active
        # tokens, scores and top-16.
        dict(name="block-f32-1", kind="block", dtype="f32", d_model=768, heads=12, head_dim=64,
             d_mlp=3072, layers=1, batch=1, n_tokens=320, a_lo=32, a_hi=32, gen=16, k_top=16),
        # Cache-aware layers of one image range with ragged active sets, as
        # images at different points of their schedules give them.
        dict(name="block-ragged-64", kind="block", dtype="bf16", d_model=1024, heads=16, head_dim=64,
             d_mlp=4096, layers=4, batch=64, n_tokens=320, a_lo=9, a_hi=71, gen=9, k_top=0),
        # A sequence length that is no multiple of any tile, heads of width 80,
        # ragged sets up to the whole sequence, with scores and selection.
        dict(name="block-odd-12", kind="block", dtype="bf16", d_model=1280, heads=16, head_dim=80,
             d_mlp=5120, layers=2, batch=12, n_tokens=229, a_lo=31, a_hi=229, gen=21, k_top=19),
        # Encoding the known tokens half-way through a generation (195 rows per
        # image, not a multiple of a key tile).
        dict(name="encode-mar-l-64", kind="encode", family="mar-l", layers=4, batch=64, n_img=256,
             n_buf=64, n_known=131),
        # The sampler on one decoding step of the headline batch (4 tokens per
        # image) and on a single image's 5 tokens, where latency is everything.
        dict(name="sample-512", kind="sample", width=1280, blocks=8, d_cond=1024, rows=512, steps=100),
        dict(name="sample-5", kind="sample", width=1280, blocks=8, d_cond=1024, rows=5, steps=100),
        # Appendix B's comparison at its quoted sizes, and the concatenating
        # baseline with ragged lengths and heads of width 80.
        dict(name="attend-two-32-256", kind="attend", batch=128, heads=16, head_dim=64, n_a=32,
             n_c=256, concat=False),
        dict(name="attend-concat-45-1503", kind="attend", batch=16, heads=16, head_dim=80, n_a=45,
             n_c=1503, concat=True),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _draw(rng):
    kind = rng.choice(["decode", "decode", "block", "block", "encode", "sample", "attend"])
    fam = rng.choice(sorted(FAMILIES))
    if kind == "decode":
        c = dict(kind=kind, family=fam, layers=rng.randint(3, 8), batch=_log(rng, 1, 96),
                 n_img=rng.choice([256, 256, 225, 1024]), n_buf=rng.choice([64, 64, 32, 47]),
                 ratio_bp=rng.choice([500, 1000, 1000, 2500]))
        c["ranges"] = min(c["batch"], rng.choice([1, 2, 2, 3]))
        return c
    if kind == "block":
        f32 = rng.random() < 0.35
        d, h, dh, f = FAMILIES[fam]
        n = rng.choice([320, 320, rng.randint(65, 400), 1088])
        hi = rng.randint(2, min(n, 150))
        return dict(kind=kind, dtype="f32" if f32 else "bf16", d_model=d, heads=h, head_dim=dh, d_mlp=f,
                    layers=rng.randint(1, 2 if f32 else 4), batch=_log(rng, 1, 8 if f32 else 96),
                    n_tokens=n, a_lo=rng.randint(1, hi), a_hi=hi, gen=rng.randint(1, 24),
                    k_top=rng.choice([0, rng.randint(1, max(1, min(40, n - hi)))]))
    if kind == "encode":
        n_img = rng.choice([256, 225])
        return dict(kind=kind, family=fam, layers=rng.randint(2, 4), batch=_log(rng, 1, 96), n_img=n_img,
                    n_buf=rng.choice([64, 64, 32, 47]), n_known=rng.randint(0, n_img))
    if kind == "sample":
        return dict(kind=kind, width=rng.choice([1024, 1280, 1536]), blocks=rng.randint(3, 12),
                    d_cond=rng.choice([768, 1024, 1280]), rows=_log(rng, 1, 900),
                    steps=rng.choice([25, 50, 100]))
    return dict(kind=kind, batch=_log(rng, 1, 128), heads=rng.choice([12, 16]),
                head_dim=rng.choice([64, 64, 80]), n_a=_log(rng, 8, 256), n_c=_log(rng, 64, 2048),
                concat=rng.random() < 0.4)


def _cost(c):
    """Rough time of a pass at the card's rates; a sampling step cannot be
    shorter than its chain of dependent products."""
    w = work(c)
    t = w["bytes"] / 5e12 + w["flops"] / 0.7e15
    return max(t, c["steps"] * (2 * c["blocks"] + 4) * 8e-6) if c["kind"] == "sample" else t


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFFFFFF)


def _randn(g, *shape, std=1.0, dtype=torch.float32):
    return (torch.randn(*shape, generator=g, device=DEV) * std).to(dtype)


def _layer(g, d, f, dtype):
    """One block's parameters: weights N(0, 0.02^2) in the model's type."""
    s = 0.02
    return {"ln1_g": 1 + _randn(g, d, std=s), "ln1_b": _randn(g, d, std=s),
            "w_qkv": _randn(g, 3 * d, d, std=s, dtype=dtype), "b_qkv": _randn(g, 3 * d, std=s),
            "w_o": _randn(g, d, d, std=s, dtype=dtype), "b_o": _randn(g, d, std=s),
            "ln2_g": 1 + _randn(g, d, std=s), "ln2_b": _randn(g, d, std=s),
            "w_1": _randn(g, f, d, std=s, dtype=dtype), "b_1": _randn(g, f, std=s),
            "w_2": _randn(g, d, f, std=s, dtype=dtype), "b_2": _randn(g, d, std=s)}


def _masked(n_img):
    """Masked image tokens before each step of the cosine schedule."""
    m = [n_img]
    for t in range(1, N_STEPS):
        m.append(max(1, min(m[-1] - 1, math.floor(n_img * math.cos(math.pi * t / (2.0 * N_STEPS))))))
    return m + [0]


def _decode_steps(c):
    """The first full step of the period-3 schedule that knows enough tokens
    for the refresh sets, and the refresh count of the step after it."""
    m, n = _masked(c["n_img"]), c["n_img"] + c["n_buf"]
    for t in range(0, N_STEPS - 1, 3):
        g, cached = m[t + 1] - m[t + 2], m[t] - m[t + 1]
        k = (c["ratio_bp"] * (n - g - cached) + 5000) // 10000
        if c["n_img"] - m[t] >= k + 8:
            return t, k
    raise ValueError(c)


def _decode_cfg(c, seed):
    d, h, dh, f = FAMILIES[c["family"]]
    return workload.Config(1000, "perf", c["layers"], d, h, dh, f, c["n_img"] + c["n_buf"], c["n_buf"],
                           c["batch"], "bf16", n_steps=N_STEPS, ratio_bp=c["ratio_bp"], sel_layer=SEL,
                           full_every=3, ln_eps=EPS, seed=int(seed))


def _decode_inputs(c, seed):
    """Weights and embeddings.  Masked positions share the mask embedding, so
    their queries agree, and each image has as many known tokens whose keys
    answer them as the step refreshes: the attention of a trained model
    singles out a few tokens in the same way, and the refresh set does not
    hang on rounding."""
    d, h, dh, f = FAMILIES[c["family"]]
    g = _gen(seed)
    layers = [_layer(g, d, f, torch.bfloat16) for _ in range(c["layers"])]
    B, n_img, n = c["batch"], c["n_img"], c["n_img"] + c["n_buf"]
    cls, value = _randn(g, B, d), _randn(g, B, n_img, d)
    mask, pos = _randn(g, d, std=2.0), _randn(g, n, d)
    w = layers[SEL - 1]
    u = torch.nn.functional.layer_norm(mask, (d,), w["ln1_g"], w["ln1_b"], EPS)
    wq, wk = w["w_qkv"][:d].float(), w["w_qkv"][d:2 * d].float()
    r = wk.t().contiguous() @ (wq @ u + w["b_qkv"][:d])
    r = (r - r.mean()) / r.std()
    t0, k = _decode_steps(c)
    orders = torch.from_numpy(workload.orders(_decode_cfg(c, seed)).astype("int64")).to(DEV)
    known = n_img - _masked(n_img)[t0]
    pick = torch.rand(B, known, generator=g, device=DEV).argsort(1)[:, :k]
    at = orders[:, :known].gather(1, pick)
    value[torch.arange(B, device=DEV)[:, None], at] = 4 * r + 0.3 * _randn(g, B, k, d)
    return layers, cls, value, mask, pos, orders


def _block_inputs(c, seed):
    """Weights, embeddings, cache contents and ragged active lists, generating
    tokens (masked positions) first.  Where the call selects a refresh set, as
    many inactive tokens have cached keys that answer the mask's query, so
    that the set does not hang on rounding."""
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    g = _gen(seed)
    d, B, n, H, dh = c["d_model"], c["batch"], c["n_tokens"], c["heads"], c["head_dim"]
    layers = [_layer(g, d, c["d_mlp"], dt) for _ in range(c["layers"])]
    cls, value = _randn(g, B, d), _randn(g, B, n, d)
    mask, pos = _randn(g, d, std=2.0), _randn(g, n, d)
    kc = _randn(g, c["layers"], B, H, n, dh, dtype=dt)
    vc = _randn(g, c["layers"], B, H, n, dh, dtype=dt)
    perm = torch.rand(B, n, generator=g, device=DEV).argsort(1).int()
    size = torch.randint(c["a_lo"], c["a_hi"] + 1, (B,), generator=g, device=DEV).tolist()
    rank = (n - 1 - perm.argsort(1)).int().contiguous()
    lists = [perm[b, :size[b]] for b in range(B)]
    gen = [min(c["gen"], a) for a in size]
    if c["k_top"]:
        w = layers[0]
        u = torch.nn.functional.layer_norm(mask, (d,), w["ln1_g"], w["ln1_b"], EPS)
        q = (w["w_qkv"][:d].float() @ u + w["b_qkv"][:d]).reshape(H, 1, dh)
        q = q * (1.5 * dh ** 0.5 / q.norm(dim=2, keepdim=True))
        for b in range(B):
            at = perm[b, size[b]:size[b] + c["k_top"]].long()
            kc[0, b, :, at] = (q + 0.2 * _randn(g, H, len(at), dh)).to(dt)
    return layers, cls, value, mask, pos, rank, kc, vc, lists, gen


def _encode_inputs(c, seed):
    d, h, dh, f = FAMILIES[c["family"]]
    g = _gen(seed)
    layers = [_layer(g, d, f, torch.bfloat16) for _ in range(c["layers"])]
    B, n_img, n = c["batch"], c["n_img"], c["n_img"] + c["n_buf"]
    e = {"cls": _randn(g, B, d), "tok": _randn(g, B, n_img, 16), "w_z": _randn(g, d, 16, std=0.25),
         "b_z": _randn(g, d, std=0.02), "pe_enc": _randn(g, n, d), "ln_g": 1 + _randn(g, d, std=0.02),
         "ln_b": _randn(g, d, std=0.02), "w_de": _randn(g, d, d, std=0.02, dtype=torch.bfloat16),
         "b_de": _randn(g, d, std=0.02), "mask": _randn(g, d), "pe_dec": _randn(g, n, d)}
    order = torch.rand(B, n_img, generator=g, device=DEV).argsort(1)
    e["known"] = order[:, :c["n_known"]].sort(1).values.int().contiguous()
    e["rank"] = order.argsort(1).int().contiguous()
    return layers, e


def _sample_inputs(c, seed):
    g = _gen(seed)
    W, nb, d, M = c["width"], c["blocks"], c["d_cond"], c["rows"]
    bf, s = torch.bfloat16, 0.02
    w = {"w_t1": _randn(g, W, 256, std=s, dtype=bf), "b_t1": _randn(g, W, std=s),
         "w_t2": _randn(g, W, W, std=s, dtype=bf), "b_t2": _randn(g, W, std=s),
         "w_c": _randn(g, W, d, std=s, dtype=bf), "b_c": _randn(g, W, std=s),
         "w_in": _randn(g, W, 16, std=0.25), "b_in": _randn(g, W, std=s),
         "w_ada": _randn(g, (3 * nb + 2) * W, W, std=s, dtype=bf), "b_ada": _randn(g, (3 * nb + 2) * W, std=s),
         "w_1": _randn(g, nb, W, W, std=s, dtype=bf), "b_1": _randn(g, nb, W, std=s),
         "w_2": _randn(g, nb, W, W, std=s, dtype=bf), "b_2": _randn(g, nb, W, std=s),
         "w_out": _randn(g, 16, W, std=s), "b_out": _randn(g, 16, std=s)}
    per = min(M, 4)  # generating tokens of an image
    B, n_img, n_buf = (M + per - 1) // per, 256, 64
    tok = torch.rand(B, n_img, generator=g, device=DEV).argsort(1)[:, :per]
    b = torch.arange(B, device=DEV)[:, None]
    rows = (b * (n_img + n_buf) + n_buf + tok).reshape(-1)[:M].int().contiguous()
    out_rows = (b * n_img + tok).reshape(-1)[:M].int().contiguous()
    x = _randn(g, B, n_img + n_buf, d)
    ln_g, ln_b = 1 + _randn(g, d, std=s), _randn(g, d, std=s)
    pe = _randn(g, n_img, d)
    noise = _randn(g, c["steps"] + 1, M, 16)
    return w, x, ln_g, ln_b, pe, rows, out_rows, noise, B, n_img, n_buf


def _attend_inputs(c, seed):
    g = _gen(seed)
    B, H, dh = c["batch"], c["heads"], c["head_dim"]
    bf = torch.bfloat16
    return (_randn(g, B, c["n_a"], H * dh, dtype=bf), _randn(g, B, H, c["n_a"], dh, dtype=bf),
            _randn(g, B, H, c["n_a"], dh, dtype=bf), _randn(g, B, H, c["n_c"], dh, dtype=bf),
            _randn(g, B, H, c["n_c"], dh, dtype=bf))


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


# ------------------------------------------------------------------ prepare

def prepare(case, seed):
    return {"kind": case["kind"], "case": case, **_PREPARE[case["kind"]](case, seed)}


def _prepare_decode(c, seed):
    layers, cls, value, mask, pos, _ = _decode_inputs(c, seed)
    weights = [{k: t.float().cpu().numpy() for k, t in w.items()} for w in layers]
    eng = driver.Engine(_decode_cfg(c, seed), DEV, weights=weights, micro_batches=c["ranges"])
    eng.e_cls, eng.e_value, eng.e_mask, eng.e_pos = cls, value, mask, pos
    return {"eng": eng, "t": _decode_steps(c)[0]}


def _prepare_block(c, seed):
    layers, cls, value, mask, pos, rank, kc, vc, lists, gen = _block_inputs(c, seed)
    d, B, n = c["d_model"], c["batch"], c["n_tokens"]
    dt = binding.MARCHE_F32 if c["dtype"] == "f32" else binding.MARCHE_BF16
    model = binding.make_model(c["layers"], d, c["heads"], c["head_dim"], c["d_mlp"], n, dt, EPS)
    size = [len(a) for a in lists]
    off = torch.tensor([0] + size).cumsum(0).int().to(DEV)
    s = {"model": model, "layers": binding.make_layers(layers), "keep": (kc, vc), "cls": cls, "value": value,
         "mask": mask, "pos": pos, "rank": rank, "idx": torch.cat(lists).contiguous(), "off": off,
         "gen": torch.tensor(gen, dtype=torch.int32, device=DEV), "total": sum(size), "max": max(size),
         "gen_max": max(gen), "x": torch.empty(B, n, d, device=DEV)}
    kb, vb = torch.empty_like(kc), torch.empty_like(vc)
    s["k"], s["v"] = kb, vb
    s["cache"] = binding.kv_cache_init(model, B, kb, vb, kb.numel() * kb.element_size(), kc, vc,
                                       stream=torch.cuda.current_stream())
    s["ws_bytes"] = binding.workspace_bytes(model, B, s["total"])
    s["ws"] = _bytes(s["ws_bytes"])
    if c["k_top"]:
        s["scores"] = torch.empty(B, c["heads"], n, device=DEV)
        s["out_off"] = (torch.arange(B, device=DEV) * c["k_top"]).int()
        s["refresh"] = torch.empty(B, c["k_top"], dtype=torch.int32, device=DEV)
    return s


def _prepare_encode(c, seed):
    layers, e = _encode_inputs(c, seed)
    d, h, dh, f = FAMILIES[c["family"]]
    B, n_enc, n = c["batch"], c["n_buf"] + c["n_known"], c["n_buf"] + c["n_img"]
    bf = binding.MARCHE_BF16
    model = binding.make_model(c["layers"], d, h, dh, f, n_enc, bf, EPS)
    k = torch.empty(c["layers"] * B * n_enc * d, dtype=torch.bfloat16, device=DEV)
    v = torch.empty_like(k)
    s = {"model": model, "layers": binding.make_layers(layers), "e": e, "keep": (k, v),
         "cache": binding.KVCache(k.data_ptr(), v.data_ptr(), c["layers"], B, h, n_enc, dh, bf),
         "idx": torch.arange(n_enc, device=DEV).repeat(B).int(),
         "off": (torch.arange(B + 1, device=DEV) * n_enc).int(),
         "x_enc": torch.empty(B, n_enc, d, device=DEV), "x_dec": torch.empty(B, n, d, device=DEV)}
    s["ws_bytes"] = binding.workspace_bytes(model, B, B * n_enc)
    s["e2d_bytes"] = binding.encoder_to_decoder_workspace_bytes(B, c["n_buf"], c["n_known"], d, bf)
    s["ws"], s["e2d"] = _bytes(s["ws_bytes"]), _bytes(s["e2d_bytes"])
    return s


def _prepare_sample(c, seed):
    w, x, ln_g, ln_b, pe, rows, out_rows, noise, B, n_img, n_buf = _sample_inputs(c, seed)
    head = binding.make_head(c["width"], c["blocks"], 16, c["d_cond"], 256, binding.MARCHE_BF16, EPS)
    nb = binding.diffusion_workspace_bytes(head, c["rows"], c["steps"])
    return {"head": head, "w": binding.make_head_weights(w), "keep": w, "x": x, "ln_g": ln_g, "ln_b": ln_b,
            "pe": pe, "rows": rows, "out_rows": out_rows, "noise": noise, "n": n_img + n_buf, "n_buf": n_buf,
            "tok": torch.zeros(B, n_img, 16, device=DEV), "ws": _bytes(nb), "ws_bytes": nb}


def _prepare_attend(c, seed):
    q, ka, va, kc, vc = _attend_inputs(c, seed)
    mode = binding.MARCHE_ATTN_CONCAT if c["concat"] else binding.MARCHE_ATTN_TWO_SEGMENT
    nb = binding.attention_workspace_bytes(c["batch"], c["heads"], c["head_dim"], c["n_a"], c["n_c"],
                                           binding.MARCHE_BF16, mode)
    return {"q": q, "ka": ka, "va": va, "kc": kc, "vc": vc, "o": torch.empty_like(q), "mode": mode,
            "ws": _bytes(nb) if nb else None, "ws_bytes": nb}


_PREPARE = {"decode": _prepare_decode, "block": _prepare_block, "encode": _prepare_encode,
            "sample": _prepare_sample, "attend": _prepare_attend}


# ------------------------------------------------------------------ run

def run(state):
    return _RUN[state["kind"]](state, state["case"])


def _run_decode(s, c):
    eng, t = s["eng"], s["t"]
    eng.step(t)
    eng.step(t + 1)
    return {"x": eng.x, "k": eng.k_cache, "v": eng.v_cache, "scores": eng.scores,
            "active": eng.plans[t + 1].ca_idx}


def _run_block(s, c):
    st = torch.cuda.current_stream()
    B, n, H = c["batch"], c["n_tokens"], c["heads"]
    top = c["k_top"]
    # every second token is known
    binding.decoder_input(s["x"], s["cls"], s["value"], s["mask"], s["pos"], s["rank"], B, n, 0,
                          c["d_model"], n // 2, stream=st)
    binding.marche_step(s["model"], s["layers"], s["cache"], 0, c["layers"], B, s["x"], s["idx"], s["off"],
                        s["gen"], s["total"], s["max"], s["gen_max"], s["scores"] if top else None,
                        0 if top else -1, s["ws"], s["ws_bytes"], stream=st)
    out = {"x": s["x"], "k": s["k"], "v": s["v"]}
    if top:
        binding.select_refresh(s["scores"], H, s["idx"], s["off"], B, n, top, s["refresh"], s["out_off"],
                               stream=st)
        out.update(scores=s["scores"], refresh=s["refresh"])
    return out


def _run_encode(s, c):
    st = torch.cuda.current_stream()
    d = FAMILIES[c["family"]][0]
    e, B, n_enc = s["e"], c["batch"], c["n_buf"] + c["n_known"]
    known = e["known"] if c["n_known"] else None
    binding.encoder_input(s["x_enc"], e["cls"], e["tok"], e["w_z"], e["b_z"], e["pe_enc"], known, B,
                          c["n_buf"], c["n_img"], c["n_known"], d, 16, stream=st)
    binding.marche_step(s["model"], s["layers"], s["cache"], 0, c["layers"], B, s["x_enc"], s["idx"],
                        s["off"], None, B * n_enc, n_enc, 0, None, -1, s["ws"], s["ws_bytes"], stream=st)
    binding.encoder_to_decoder(s["x_dec"], s["x_enc"], e["ln_g"], e["ln_b"], EPS, e["w_de"], e["b_de"],
                               e["mask"], e["pe_dec"], known, e["rank"], B, c["n_buf"], c["n_img"],
                               c["n_known"], d, binding.MARCHE_BF16, s["e2d"], s["e2d_bytes"], stream=st)
    return {"x_enc": s["x_enc"], "x_dec": s["x_dec"]}


def _run_sample(s, c):
    binding.diffusion_sample(s["head"], s["w"], s["x"], s["n"], s["n_buf"], s["ln_g"], s["ln_b"], EPS,
                             s["pe"], s["rows"], s["out_rows"], c["rows"], s["noise"], c["steps"], 1.0,
                             s["tok"], s["ws"], s["ws_bytes"], stream=torch.cuda.current_stream())
    return s["tok"]


def _run_attend(s, c):
    binding.attention_segments(s["q"], s["o"], c["n_a"], s["ka"], s["va"], c["n_a"], s["kc"], s["vc"],
                               c["n_c"], c["batch"], c["heads"], c["head_dim"], binding.MARCHE_BF16,
                               s["mode"], s["ws"], s["ws_bytes"], stream=torch.cuda.current_stream())
    return s["o"]


_RUN = {"decode": _run_decode, "block": _run_block, "encode": _run_encode, "sample": _run_sample,
        "attend": _run_attend}


# ------------------------------------------------------------------ work and tolerance

def _layers_work(rows, images, n, d, f, layers, es):
    """Block layers on `rows` active rows of `images` images of n tokens:
    weights, the cache and x each once."""
    wt = layers * (4 * d * d + 2 * d * f)
    flops = 2.0 * rows * wt + 4.0 * layers * rows * n * d
    return es * (wt + layers * 2.0 * images * n * d) + 8.0 * rows * d, flops


def work(case):
    c = case
    if c["kind"] == "decode":
        d, h, dh, f = FAMILIES[c["family"]]
        n, B, L = c["n_img"] + c["n_buf"], c["batch"], c["layers"]
        t0, k = _decode_steps(c)
        m = _masked(c["n_img"])
        a = (m[t0] - m[t0 + 1]) + (m[t0 + 1] - m[t0 + 2]) + k
        b1, f1 = _layers_work(B * n, B, n, d, f, L, 2)
        b2, f2 = _layers_work(B * n, B, n, d, f, SEL, 2)
        b3, f3 = _layers_work(B * a, B, n, d, f, L - SEL, 2)
        return {"bytes": b1 + b2 + b3 + 4.0 * B * n * d, "flops": f1 + f2 + f3}
    if c["kind"] == "block":
        d, B, n = c["d_model"], c["batch"], c["n_tokens"]
        rows = B * (c["a_lo"] + c["a_hi"]) / 2
        es = 4 if c["dtype"] == "f32" else 2
        b, f = _layers_work(rows, B, n, d, c["d_mlp"], c["layers"], es)
        return {"bytes": b + 4.0 * (1.5 * B * n * d + n * d), "flops": f}
    if c["kind"] == "encode":
        d, h, dh, f = FAMILIES[c["family"]]
        n, n_enc, B = c["n_img"] + c["n_buf"], c["n_buf"] + c["n_known"], c["batch"]
        b, fl = _layers_work(B * n_enc, B, n_enc, d, f, c["layers"], 2)
        return {"bytes": b + 2.0 * d * d + 4.0 * (B * n * d + 2 * n * d), "flops": fl + 2.0 * B * n_enc * d * (d + 16)}
    if c["kind"] == "sample":
        W, nb, M, T, d = c["width"], c["blocks"], c["rows"], c["steps"], c["d_cond"]
        wt = (3 * nb + 2) * W * W + 2 * nb * W * W
        return {"bytes": 2.0 * (wt + W * (256 + W + d)) + 4.0 * ((T + 1) * M * 16 + M * d + 2 * W * 16),
                "flops": 2.0 * T * M * (wt + 32 * W) + 2.0 * M * W * d + 2.0 * T * W * (256 + W)}
    B, H, dh, na, nc = c["batch"], c["heads"], c["head_dim"], c["n_a"], c["n_c"]
    return {"bytes": 4.0 * B * H * dh * (na + na + nc), "flops": 4.0 * B * H * na * (na + nc) * dh}


def tolerance(case):
    """About four times the distance from ``exact``: up to 2.6e-3 with bf16
    activations, weights and cache, 1.2e-7 in fp32 (where sums in another
    order move a value by up to about 1e-6)."""
    if case["kind"] == "block" and case["dtype"] == "f32":
        return {"rel": 2e-6, "differ": 0.0}
    return {"rel": 0.01, "differ": 0.01}


# ------------------------------------------------------------------ float64 reference

def _ln64(x, g=None, b=None):
    x = x - x.mean(-1, keepdim=True)
    x = x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)
    return x if g is None else x * g + b


def _block64(w, x, k, v, rows, heads, n_gen=0):
    """One block on the active rows of a group of images with equally long
    lists: x [B][N][D], k / v [B][H][N][dh] (updated in place), rows [B][a].
    Returns the per-head attention mass of the first n_gen rows."""
    B, n, d = x.shape
    a = rows.shape[1]
    dh = d // heads
    at = rows[:, :, None].expand(B, a, d)
    xa = x.gather(1, at)
    qkv = _ln64(xa, w["ln1_g"], w["ln1_b"]) @ w["w_qkv"].t().contiguous() + w["b_qkv"]
    q, kn, vn = (t.reshape(B, a, heads, dh).transpose(1, 2).contiguous() for t in qkv.split(d, -1))
    cols = rows[:, None, :, None].expand(B, heads, a, dh)
    k.scatter_(2, cols, kn)
    v.scatter_(2, cols, vn)
    p = torch.softmax(q @ k.transpose(-1, -2).contiguous() / math.sqrt(dh), -1)
    o = (p @ v).transpose(1, 2).reshape(B, a, d)
    xa = xa + o @ w["w_o"].t().contiguous() + w["b_o"]
    hid = torch.nn.functional.gelu(_ln64(xa, w["ln2_g"], w["ln2_b"]) @ w["w_1"].t().contiguous() + w["b_1"])
    xa = xa + hid @ w["w_2"].t().contiguous() + w["b_2"]
    x.scatter_(1, at, xa)
    return p[:, :, :n_gen].sum(2) if n_gen else None


def _f64(w):
    return {k: t.double() for k, t in w.items()}


def exact(case, seed):
    return _EXACT[case["kind"]](case, seed)


def _exact_decode(c, seed):
    layers, cls, value, mask, pos, orders = _decode_inputs(c, seed)
    layers = [_f64(w) for w in layers]
    cls, value, mask, pos = (t.double() for t in (cls, value, mask, pos))
    d, H, dh, _ = FAMILIES[c["family"]]
    B, n_img, nb, L = c["batch"], c["n_img"], c["n_buf"], c["layers"]
    n = n_img + nb
    m = _masked(n_img)
    t0, k_ref = _decode_steps(c)
    rank = orders.argsort(1)
    x = torch.empty(B, n, d, dtype=torch.float64, device=DEV)
    K = torch.zeros(L, B, H, n, dh, dtype=torch.float64, device=DEV)
    V = torch.zeros_like(K)
    S = torch.empty(B, H, n, dtype=torch.float64, device=DEV)
    chunk = max(1, min(B, int(1.5e8 // (H * n * n))))
    for b0 in range(0, B, chunk):
        sl = slice(b0, min(B, b0 + chunk))
        nbat = sl.stop - sl.start
        for t in (t0, t0 + 1):
            known = n_img - m[t]
            img = torch.where((rank[sl] < known)[:, :, None], value[sl], mask)
            xs = pos + torch.cat([cls[sl][:, None].expand(nbat, nb, d), img], 1)
            gen = orders[sl, known:n_img - m[t + 1]] + nb
            rest = torch.ones(nbat, n, dtype=torch.bool, device=DEV).scatter_(1, gen, False)
            tok = torch.arange(n, device=DEV).expand(nbat, n)
            rows = torch.cat([gen, tok[rest].reshape(nbat, -1)], 1)
            full = t == t0
            for l in range(L if full else SEL):
                s = _block64(layers[l], xs, K[l, sl], V[l, sl], rows, H,
                             gen.shape[1] if not full and l == SEL - 1 else 0)
            if not full:
                S[sl] = s
                lead = torch.cat([gen, orders[sl, n_img - m[t - 1]:known] + nb], 1)
                pick = s.sum(1).scatter(1, lead, -math.inf).topk(k_ref, 1).indices.sort(1).values
                rows = torch.cat([lead, pick], 1)
                for l in range(SEL, L):
                    _block64(layers[l], xs, K[l, sl], V[l, sl], rows, H)
        x[sl] = xs
    return {"x": x, "k": K.reshape(-1), "v": V.reshape(-1), "scores": S, "active": None}


def _exact_block(c, seed):
    layers, cls, value, mask, pos, rank, kc, vc, lists, gen = _block_inputs(c, seed)
    B, n, H = c["batch"], c["n_tokens"], c["heads"]
    x = pos.double() + torch.where((rank < n // 2)[:, :, None], value.double(), mask.double())
    K, V = kc.double(), vc.double()
    S = torch.empty(B, H, n, dtype=torch.float64, device=DEV)
    for l, w in enumerate(layers):
        w = _f64(w)
        for b in range(B):
            xb = x[b:b + 1]
            s = _block64(w, xb, K[l, b:b + 1], V[l, b:b + 1], lists[b][None].long(), H,
                         gen[b] if c["k_top"] and l == 0 else 0)
            if s is not None:
                S[b] = s[0]
    out = {"x": x, "k": K, "v": V}
    if c["k_top"]:
        out.update(scores=S, refresh=None)
    return out


def _exact_encode(c, seed):
    layers, e = _encode_inputs(c, seed)
    e = {k: t if t.dtype == torch.int32 else t.double() for k, t in e.items()}
    d, H, dh, _ = FAMILIES[c["family"]]
    B, nb, nk = c["batch"], c["n_buf"], c["n_known"]
    n_enc, n = nb + nk, nb + c["n_img"]
    known = e["known"].long()
    tok = e["tok"].gather(1, known[:, :, None].expand(B, nk, 16))
    x = torch.cat([e["cls"][:, None] + e["pe_enc"][:nb],
                   tok @ e["w_z"].t().contiguous() + e["b_z"] + e["pe_enc"][nb + known]], 1)
    rows = torch.arange(n_enc, device=DEV).expand(B, n_enc)
    K = torch.zeros(B, H, n_enc, dh, dtype=torch.float64, device=DEV)
    V = torch.zeros_like(K)
    for w in layers:
        _block64(_f64(w), x, K, V, rows, H)
    v = _ln64(x, e["ln_g"], e["ln_b"]) @ e["w_de"].t().contiguous() + e["b_de"]
    y = (e["mask"] + e["pe_dec"]).repeat(B, 1, 1)
    at = torch.cat([torch.arange(nb, device=DEV).expand(B, nb), nb + known], 1)
    y.scatter_(1, at[:, :, None].expand(B, n_enc, d), v + e["pe_dec"][at])
    return {"x_enc": x, "x_dec": y}


def _exact_sample(c, seed):
    w, x, ln_g, ln_b, pe, rows, out_rows, noise, B, n_img, n_buf = _sample_inputs(c, seed)
    w = _f64(w)
    W, nb, T = c["width"], c["blocks"], c["steps"]
    rows, out_rows = rows.long(), out_rows.long()
    silu = torch.nn.functional.silu
    z = _ln64(x.reshape(-1, c["d_cond"])[rows].double(), ln_g.double(), ln_b.double())
    z = z + pe.double()[rows % (n_img + n_buf) - n_buf]
    freq = torch.exp(-math.log(10000.0) * torch.arange(128, dtype=torch.float64, device=DEV) / 128)
    arg = torch.arange(T, dtype=torch.float64, device=DEV)[:, None] * freq
    wt = {k: w[k].transpose(-1, -2).contiguous() for k in ("w_t1", "w_t2", "w_c", "w_in", "w_ada", "w_1", "w_2", "w_out")}
    temb = silu(torch.cat([arg.cos(), arg.sin()], 1) @ wt["w_t1"] + w["b_t1"]) @ wt["w_t2"] + w["b_t2"]
    cond = z @ wt["w_c"] + w["b_c"]
    curve = [math.cos((i / T + 0.008) / 1.008 * math.pi / 2) ** 2 for i in range(T + 1)]
    beta = [min(1 - curve[i + 1] / curve[i], 0.999) for i in range(T)]
    bar = [1.0]
    for b in beta:
        bar.append(bar[-1] * (1 - b))
    noise = noise.double()
    tok = noise[T]
    for i in range(T - 1, -1, -1):
        mod = silu(cond + temb[i]) @ wt["w_ada"] + w["b_ada"]
        s = mod.split(W, -1)
        h = tok @ wt["w_in"] + w["b_in"]
        for k in range(nb):
            a = _ln64(h) * (1 + s[3 * k + 1]) + s[3 * k]
            h = h + s[3 * k + 2] * (silu(a @ wt["w_1"][k] + w["b_1"][k]) @ wt["w_2"][k] + w["b_2"][k])
        eps = (_ln64(h) * (1 + s[3 * nb + 1]) + s[3 * nb]) @ wt["w_out"] + w["b_out"]
        ab, prev, b = bar[i + 1], bar[i], beta[i]
        x0 = (tok - math.sqrt(1 - ab) * eps) / math.sqrt(ab)
        tok = b * math.sqrt(prev) / (1 - ab) * x0 + (1 - prev) * math.sqrt(1 - b) / (1 - ab) * tok
        if i:
            tok = tok + math.sqrt(b * (1 - prev) / (1 - ab)) * noise[i]
    out = torch.zeros(B * n_img, 16, dtype=torch.float64, device=DEV)
    out[out_rows] = tok
    return out.reshape(B, n_img, 16)


def _exact_attend(c, seed):
    q, ka, va, kc, vc = _attend_inputs(c, seed)
    B, H, dh, na = c["batch"], c["heads"], c["head_dim"], c["n_a"]
    out = torch.empty(B, na, H * dh, dtype=torch.float64, device=DEV)
    for b in range(B):
        k = torch.cat([ka[b], kc[b]], 1).double()
        v = torch.cat([va[b], vc[b]], 1).double()
        p = torch.softmax(q[b].double().reshape(na, H, dh).transpose(0, 1).contiguous()
                          @ k.transpose(1, 2).contiguous() / math.sqrt(dh), -1)
        out[b] = (p @ v).transpose(0, 1).reshape(na, H * dh)
    return out


_EXACT = {"decode": _exact_decode, "block": _exact_block, "encode": _exact_encode,
          "sample": _exact_sample, "attend": _exact_attend}
