"""One block at the edges of the launch rules, against the fp64 oracle: fp32
products of one row, of 16 / 32 / 64-row remainders and of enough rows for the
64x64 tile; fp32 attention with one and with four rows per workgroup; bf16
attention on ragged key tails at both head widths for one to four query
blocks, with the score pass as a kernel of its own, and stand-alone with few
(image, head) pairs (two key groups per workgroup) and with many; the tiles of
32, 64, 192 and 256 rows with ragged last tiles; the sampler's block
products and modulations at the row counts where their kernels change; the
encoder input at its channel widths, with one row per wavefront and several."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import mar
from paper_2506_12035_amd import workload
from tests.gpu_util import TOL, SingleLayer, f64, rel_err, say
from tests.test_gpu_layer import _check_layer, _oracle_layer
from tests.test_gpu_mar import _oracle_head, _run_head

pytestmark = pytest.mark.gpu


def _case(cfg, sizes, gens, seed):
    rng = np.random.default_rng(seed)
    B, N = len(sizes), cfg.n_tokens
    x = rng.standard_normal((B, N, cfg.d_model), dtype=np.float32)
    kv = [workload.round_to(rng.standard_normal((B, cfg.n_heads, N, cfg.head_dim), dtype=np.float32),
                            cfg.dtype) for _ in range(2)]
    active = [rng.permutation(N)[:s].astype(np.int32) for s in sizes]
    p = workload.layer_weights(cfg, 0)
    say(f"{cfg.name} N={N} sizes={sizes[:6]}.. gens={gens[:6]}..")
    ref = _oracle_layer(cfg, f64(p), x, *kv, active, gens)
    gpu = SingleLayer(cfg, p, x, *kv).run(active, gens)
    _check_layer(cfg, x, *kv, active, gens, gpu, ref, TOL[cfg.dtype])


# (d_model, heads, head_dim, N, active rows per image, generating rows).  Eight
# images of 190 rows give M = 1335: the 64x64 tile at N = 768 and 1024 columns,
# the skinny kernel at 256, and four rows per workgroup in the attention.
F32 = [
    (256, 4, 64, 37, [1], [1]),
    (256, 4, 64, 65, [17], [3]),
    (768, 12, 64, 130, [32, 1], [17, 1]),
    (1280, 16, 80, 71, [33, 32, 6], [20, 1, 6]),
    (256, 4, 64, 190, [190] * 7 + [5], [9] * 7 + [5]),
    (1280, 16, 80, 203, [203, 40, 80], [2, 40, 16]),
]


@pytest.mark.parametrize("case", F32, ids=lambda c: f"d{c[0]}h{c[2]}n{c[3]}m{sum(c[4])}")
def test_f32_layer_shapes(case):
    d, h, dh, n, sizes, gens = case
    cfg = workload.Config(60, "f32-shape", 1, d, h, dh, 4 * d, n, 0, len(sizes), "f32")
    _case(cfg, sizes, gens, seed=sum(sizes) + n)


# Lists up to 32, 64, 128 and more rows; key tails of 1 and 37, and aligned
# lengths.  More than 64 generating rows need the separate score pass at every
# length that the resident kernel does not take.
BF16 = [
    (1024, 16, 64, 65, [32, 5], [32, 2]),
    (1024, 16, 64, 229, [64, 33], [9, 33]),
    (1024, 16, 64, 192, [100, 3], [70, 3]),
    (1280, 16, 80, 101, [31, 1], [31, 1]),
    (1280, 16, 80, 449, [129, 64], [80, 5]),
    (1024, 16, 64, 357, [32, 1, 7, 32, 3, 9, 30, 2, 31], [3] * 1 + [1] * 8),
    (1280, 16, 80, 320, [32, 1, 7, 32, 3, 9, 30, 2, 31], [3] * 1 + [1] * 8),
    (1280, 16, 80, 357, [64, 33, 40, 1, 2, 64, 50, 12, 9], [7] * 3 + [1] * 6),
    (1024, 16, 64, 293, [128, 65, 96, 1, 97, 33, 50, 128, 9], [70] + [1] * 8),
    (1024, 16, 64, 320, [128, 65, 96, 1, 97, 33, 50, 128, 9], [70] + [1] * 8),
]


@pytest.mark.parametrize("case", BF16, ids=lambda c: f"h{c[2]}n{c[3]}b{len(c[4])}a{max(c[4])}")
def test_bf16_attention_shapes(case):
    d, h, dh, n, sizes, gens = case
    cfg = workload.Config(61, "bf16-shape", 1, d, h, dh, 1024, n, 0, len(sizes), "bf16")
    _case(cfg, sizes, gens, seed=sum(sizes) + n)


# 65 to 128 rows with scores: (d_model, heads, head_dim, N, rows, generating rows,
# the attention kernel that writes the scores).  The resident one where the
# streaming one cannot (heads of 80, a key tail, over 64 generating rows).
SCORES = [
    (1280, 16, 80, 320, [65, 3], [9, 3], "attention_res_scores_ca"),
    (1280, 16, 80, 229, [128, 70], [66, 1], "attention_res_scores_ca"),
    (1024, 16, 64, 289, [100, 1], [33, 1], "attention_res_scores_ca"),
    (1024, 16, 64, 128, [66, 20], [5, 20], "attention_res_scores_ca"),
    (1024, 16, 64, 320, [128, 9], [65, 9], "attention_res_scores_ca"),
    (1024, 16, 64, 320, [128, 9], [64, 9], "attention_scores_ca"),
    (1280, 16, 80, 320, [64, 3], [9, 3], "attn_scores_ca"),
]


@pytest.mark.parametrize("case", SCORES, ids=lambda c: f"h{c[2]}n{c[3]}a{max(c[4])}g{max(c[5])}")
def test_score_layers_of_65_to_128_rows(case):
    from paper_2506_12035_amd import binding

    d, h, dh, n, sizes, gens, kernel = case
    cfg = workload.Config(64, "score-rows", 1, d, h, dh, 1024, n, 0, len(sizes), "bf16")
    binding.profile_reset()
    binding.profile_enable(True)
    try:
        _case(cfg, sizes, gens, seed=sum(sizes) + n)
        prof = binding.profile_collect()
    finally:
        binding.profile_enable(False)
        binding.profile_reset()
    assert kernel in prof, sorted(prof)


# (dtype, d_model, heads, head_dim, N, active rows): the streaming kernels with one
# to four query blocks and the resident one, with the scores inside, and a score
# pass of its own.
EMPTY = [
    ("bf16", 1024, 16, 64, 320, [30, 0, 7]), ("bf16", 1024, 16, 64, 320, [0, 64]),
    ("bf16", 1024, 16, 64, 384, [128, 0]), ("bf16", 1024, 16, 64, 384, [200, 0]),
    ("bf16", 1024, 16, 64, 320, [0, 200, 0]), ("bf16", 1280, 16, 80, 229, [100, 0]),
    ("bf16", 1280, 16, 80, 229, [40, 0]), ("f32", 256, 4, 64, 130, [0, 20]),
]


@pytest.mark.parametrize("case", EMPTY, ids=lambda c: "{}h{}n{}-{}".format(c[0], c[3], c[4], "-".join(map(str, c[5]))))
def test_image_without_active_rows(case):
    """Its scores are 0 (the buffer held NaN) and its rows stay; the others'
    are those of a call without it."""
    dtype, d, h, dh, n, sizes = case
    cfg = workload.Config(66, "empty", 1, d, h, dh, 512, n, 0, len(sizes), dtype)
    say(f"empty images: {dtype} dh={dh} N={n} sizes={sizes}")
    rng = np.random.default_rng(n + sum(sizes))
    B = len(sizes)
    x = rng.standard_normal((B, n, d), dtype=np.float32)
    k, v = (workload.round_to(rng.standard_normal((B, h, n, dh), dtype=np.float32), dtype) for _ in range(2))
    act = [rng.permutation(n)[:s].astype(np.int32) for s in sizes]
    gens = [min(3, s) for s in sizes]
    p = workload.layer_weights(cfg, 0)
    got = SingleLayer(cfg, p, x, k, v).run(act, gens)
    live = [b for b in range(B) if sizes[b]]
    ref = SingleLayer(cfg, p, x[live], k[live], v[live]).run([act[b] for b in live], [gens[b] for b in live])
    for name in ("x", "k", "v", "scores"):
        assert np.array_equal(got[name][live], ref[name]), name
    for b in set(range(B)) - set(live):
        assert np.array_equal(got["x"][b], x[b]) and not got["scores"][b].any(), b


# Active rows per image at D = 1024, MLP 4096, and a tile each product count
# takes: 192 rows x 128 columns with 135 rows in the last tile, 256 x 128 with
# one, 192 x 128 over several rounds of N = 1024; and the tiles of a few rows,
# with one row in the last tile of 32 and 33 in the last of 64.
TILES = [
    ([96, 1], {"gemm_qkv_t64x64_ca", "gemm_o_t32x64_ca", "gemm_fc2_t32x32_ca"}),
    ([1], {"gemm_qkv_t32x64_ca", "gemm_o_t32x32_ca"}),
    ([320] * 4 + [7], {"gemm_fc1_t192x128_ca"}),
    ([320] * 7 + [65], {"gemm_qkv_t256x128_ca"}),
    ([320] * 12 + [320, 1], {"gemm_o_t192x128_ca", "gemm_fc2_t192x128_ca"}),
]


@pytest.mark.parametrize("sizes,classes", TILES, ids=lambda v: str(sum(v)) if isinstance(v, list) else "")
def test_gemm_tile_edges(sizes, classes):
    from paper_2506_12035_amd import binding

    cfg = workload.Config(62, "tile-edge", 1, 1024, 16, 64, 4096, 320, 0, len(sizes), "bf16")
    binding.profile_reset()
    binding.profile_enable(True)
    try:
        _case(cfg, sizes, [1] * len(sizes), seed=sum(sizes))
        prof = binding.profile_collect()
    finally:
        binding.profile_enable(False)
        binding.profile_reset()
    assert classes <= set(prof), sorted(prof)


# (batch, heads, head_dim, queries, active keys, cached keys).  One and two key
# groups; segments shorter than a tile, of one key, of whole tiles, and a
# single segment; queries that are not the active keys.
SEGMENTS = [
    (2, 4, 64, 1, 1, 63), (2, 4, 80, 32, 64, 1), (3, 4, 80, 33, 1, 130), (2, 4, 64, 64, 0, 320),
    (1, 4, 64, 200, 65, 128), (33, 8, 64, 17, 17, 47), (33, 8, 80, 40, 3, 190),
    (22, 12, 64, 100, 64, 64), (22, 12, 80, 129, 100, 1),
]


@pytest.mark.parametrize("case", SEGMENTS, ids=lambda c: "b{}h{}d{}q{}-{}-{}".format(*c))
def test_segment_shapes(case):
    import torch
    from oracle import block
    from paper_2506_12035_amd import binding

    B, H, dh, nq, na, nc = case
    say(f"segment attention {case}")
    rng = np.random.default_rng(nq + na + nc)
    draw = lambda *s: workload.round_to(rng.standard_normal(s, dtype=np.float32), "bf16")
    q, ka, va, kc, vc = (draw(B, nq, H * dh), draw(B, H, na, dh), draw(B, H, na, dh),
                         draw(B, H, nc, dh), draw(B, H, nc, dh))
    dev = [torch.from_numpy(t).to("cuda").bfloat16() if t.size else None for t in (q, ka, va, kc, vc)]
    o = torch.full((B, nq, H * dh), float("nan"), device="cuda", dtype=torch.bfloat16)
    binding.attention_segments(dev[0], o, nq, dev[1], dev[2], na, dev[3], dev[4], nc, B, H, dh,
                               binding.MARCHE_BF16, binding.MARCHE_ATTN_TWO_SEGMENT)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy().reshape(B, nq, H, dh)
    for b in (0, B - 1):
        for h in range(H):
            ref = block.attention_two_segment(q[b, :, h * dh:(h + 1) * dh], ka[b, h], va[b, h],
                                              kc[b, h], vc[b, h])
            assert rel_err(got[b, :, h], ref) <= TOL["bf16"], (b, h)


@pytest.mark.parametrize("dead", ["cached"])
@pytest.mark.parametrize("B,dh,nq", [(1, 64, 20), (1, 80, 50), (20, 64, 50), (20, 80, 20), (6, 64, 140)])
def test_infinite_keys_of_a_segment(B, dh, nq, dead):
    """A segment whose keys all lie at -inf from every query has no weight: the
    result is that of the other segment (both 64 keys, so that a segment is a
    key tile, with few workgroups a key group's only one)."""
    import torch
    from oracle import block
    from paper_2506_12035_amd import binding

    H, n = 16, 64
    say(f"infinite {dead} keys: B={B} dh={dh} nq={nq}")
    rng = np.random.default_rng(nq)
    draw = lambda *s: workload.round_to(rng.standard_normal(s, dtype=np.float32), "bf16")
    q, ka, va, kc, vc = draw(B, nq, H * dh), *(draw(B, H, n, dh) for _ in range(4))
    q[:, :, ::dh] = np.abs(q[:, :, ::dh]) + 0.25
    (kc if dead == "cached" else ka)[..., 0] = -np.inf
    dev = [torch.from_numpy(t).to("cuda").bfloat16() for t in (q, ka, va, kc, vc)]
    o = torch.full((B, nq, H * dh), float("nan"), device="cuda", dtype=torch.bfloat16)
    binding.attention_segments(dev[0], o, nq, dev[1], dev[2], n, dev[3], dev[4], n, B, H, dh,
                               binding.MARCHE_BF16, binding.MARCHE_ATTN_TWO_SEGMENT)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy().reshape(B, nq, H, dh)
    k, v = (ka, va) if dead == "cached" else (kc, vc)
    for h in range(H):
        ref = block.attention(q[-1, :, h * dh:(h + 1) * dh], k[-1, h], v[-1, h])[0]
        assert rel_err(got[-1, :, h], ref) <= TOL["bf16"], h


# (rows, width, blocks, sampling steps, channels, dtype, kernel of the block
# products): the few-row kernel with one, two and three blocks of 16 rows ("norm":
# forming the modulated norm itself, up to 8 rows, from width 1536 on up to 16 as
# far as they fit) up to the last row count and the widest launches it takes, the next row or width on a tile; the
# 32x64, 64x64 and 64x128 tiles with side products and a ragged last tile; row
# counts whose modulations no longer fit beside the block products; one block
# (no side products) and more, one to three sampling steps, other channel counts.
SAMPLER = [
    (1, 256, 2, 3, 16, "bf16", "norm"),
    (8, 1280, 2, 2, 16, "bf16", "norm"),
    (9, 1280, 2, 2, 16, "bf16", "rows"),
    (16, 512, 3, 2, 16, "bf16", "rows"),
    (9, 1536, 1, 2, 8, "bf16", "rows"),
    (16, 1536, 3, 2, 16, "bf16", "norm"),
    (17, 1536, 3, 2, 16, "bf16", "t32x64"),
    (16, 2048, 2, 2, 16, "bf16", "rows"),
    (5, 4096, 2, 1, 16, "bf16", "t32x64"),
    (17, 256, 1, 3, 5, "bf16", "rows"),
    (33, 768, 2, 1, 16, "bf16", "rows"),
    (48, 1024, 3, 2, 16, "bf16", "rows"),
    (49, 1024, 3, 2, 16, "bf16", "t32x64"),
    (64, 256, 5, 3, 33, "bf16", "t32x64"),
    (65, 512, 2, 3, 16, "bf16", "t32x64"),
    (200, 1024, 2, 2, 16, "bf16", "t64x64"),
    (300, 1024, 2, 2, 16, "bf16", "t64x128"),
    (200, 256, 1, 2, 16, "bf16", "t32x64"),
    (1500, 1280, 3, 2, 16, "bf16", "t64x128"),
    (5, 256, 2, 3, 16, "f32", None),
    (70, 512, 1, 2, 3, "f32", None),
]


@pytest.mark.parametrize("case", SAMPLER, ids=lambda c: "m{}w{}n{}t{}c{}-{}".format(*c))
def test_sampler_shapes(case):
    from paper_2506_12035_amd import binding

    rows, width, blocks, steps, chans, dtype, kernel = case
    tiny = workload.MAR_CONFIGS["tiny"]
    B = rows // 100 + 2
    mc = replace(tiny, dec=tiny.dec.with_(dtype=dtype, n_tokens=104, batch=B), head_width=width,
                 head_blocks=blocks, sample_steps=steps, c_tok=chans, head_std=0.04)
    cfg = mc.dec
    say(f"sampler rows={rows} width={width} blocks={blocks} steps={steps} channels={chans} {dtype}")
    hs = mar.HeadShape(width, blocks, chans, cfg.d_model, mc.t_freq, mc.head_eps)
    head, emb = workload.head_weights(mc), workload.mar_embeddings(mc)
    rng = np.random.default_rng(rows + width)
    x_dec = rng.standard_normal((B, cfg.n_tokens, cfg.d_model)).astype(np.float32)
    cells = rng.choice(B * cfg.n_img, size=rows, replace=False)
    b_of, p_of = cells // cfg.n_img, cells % cfg.n_img
    out_rows = (b_of * cfg.n_img + p_of).astype(np.int32)
    src = (b_of * cfg.n_tokens + cfg.n_buf + p_of).astype(np.int32)
    noise = workload.head_noise(mc, rows, rows)
    binding.profile_reset()
    binding.profile_enable(True)
    try:
        got = _run_head(mc, head, emb, x_dec, src, out_rows, noise, 1.0)
        prof = binding.profile_collect()
    finally:
        binding.profile_enable(False)
        binding.profile_reset()
    if kernel and blocks > 1:
        assert ("head_mod" in prof) == (kernel != "norm"), sorted(prof)
    if kernel:
        kernel = "rows" if kernel == "norm" else kernel
        assert {f"gemm_head_silu_{kernel}", f"gemm_head_{kernel}"} <= set(prof), sorted(prof)
    ref = _oracle_head(mc, hs, head, emb, x_dec, b_of, p_of, noise, 1.0)
    e = rel_err(got[out_rows], ref)
    say(f"  max rel err {e:.2e}")
    assert e <= TOL[dtype]
    assert np.isnan(got[np.setdiff1d(np.arange(got.shape[0]), out_rows)]).all()


# (width, blocks, channels, dtype, rows of the whole call, rows of its parts): parts
# on every kernel that a row count picks (norm inside the first product, one to
# three row blocks of the few-row kernel, the 32x64, 64x64 and 64x128 tiles, with
# and without side products), fp32 on both sides of the 64x64 tile.
SAMPLER_PARTS = [
    (256, 3, 16, "bf16", 300, [1, 16, 17, 33, 48, 49, 130]),
    (1024, 3, 16, "bf16", 700, [1, 5, 15, 16, 17, 31, 40, 48, 49, 65, 129, 300]),
    (2048, 2, 4, "bf16", 130, [2, 13, 14, 16, 17, 40]),
    (1280, 2, 16, "bf16", 60, [8, 9]),
    (1280, 1, 16, "bf16", 200, [3, 16, 20, 35, 60]),
    (512, 2, 33, "f32", 1500, [1, 17, 40, 300]),
]


@pytest.mark.parametrize("case", SAMPLER_PARTS, ids=lambda c: "w{}n{}c{}-{}-m{}".format(*c))
def test_sampler_rows_do_not_depend_on_the_call(case):
    """The first rows of a call, sampled in a call of their own: bit for bit
    the same values, whichever kernels the two row counts take."""
    width, blocks, chans, dtype, rows, parts = case
    tiny = workload.MAR_CONFIGS["tiny"]
    B = rows // 100 + 2
    mc = replace(tiny, dec=tiny.dec.with_(dtype=dtype, n_tokens=104, batch=B), head_width=width,
                 head_blocks=blocks, sample_steps=3, c_tok=chans, head_std=0.04)
    cfg = mc.dec
    head, emb = workload.head_weights(mc), workload.mar_embeddings(mc)
    rng = np.random.default_rng(rows + width)
    x_dec = rng.standard_normal((B, cfg.n_tokens, cfg.d_model)).astype(np.float32)
    cells = rng.choice(B * cfg.n_img, size=rows, replace=False)
    out_rows = cells.astype(np.int32)
    src = (cells // cfg.n_img * cfg.n_tokens + cfg.n_buf + cells % cfg.n_img).astype(np.int32)
    noise = workload.head_noise(mc, rows, rows)
    whole = _run_head(mc, head, emb, x_dec, src, out_rows, noise, 1.0)
    for m in parts:
        say(f"sampler width={width} {dtype}: {m} of {rows} rows")
        got = _run_head(mc, head, emb, x_dec, src[:m], out_rows[:m],
                        np.ascontiguousarray(noise[:, :m]), 1.0)
        assert np.array_equal(got[out_rows[:m]], whole[out_rows[:m]]), m


# (images, n_buf, n_img, n_known, d_model, channels).  64 images of 157 rows
# give a wavefront five to ten rows of 512 columns (the last group ragged,
# buffer and image rows within one group), two images one row; the channels sit
# on both sides of each compile-time width.
ENC_IN = [
    (64, 7, 200, 150, 512, 16),
    (64, 7, 200, 150, 512, 64),
    (64, 7, 200, 150, 256, 33),
    (2, 3, 20, 11, 1280, 17),
    (2, 0, 20, 20, 256, 5),
    (2, 3, 20, 11, 4096, 1),
]


@pytest.mark.parametrize("B,n_buf,n_img,n_known,D,C", ENC_IN)
def test_encoder_input_rows(B, n_buf, n_img, n_known, D, C):
    """Within 1e-6 of the largest output: a sum of at most 64 products in fp32
    is off by 64 x 2^-24 of its terms' size, an order below that of a row's
    largest output here.  The weights start at an odd word: they need 4-byte
    alignment only."""
    import torch

    from paper_2506_12035_amd import binding

    say(f"encoder input B={B} n_buf={n_buf} n_known={n_known} D={D} C={C}")
    rng = np.random.default_rng(7)
    cls, tok, b_z, pe, w_z = (rng.standard_normal(s).astype(np.float32) for s in (
        (B, D), (B, n_img, C), (D,), (n_buf + n_img, D), (D, C)))
    w_z *= 0.25
    known = np.stack([np.sort(rng.permutation(n_img)[:n_known]) for _ in range(B)]).astype(np.int32)
    dev = [torch.from_numpy(a).cuda() for a in (cls, tok, b_z, pe, known)]
    w_dev = torch.empty(D * C + 1, device="cuda")[1:].view(D, C)
    w_dev.copy_(torch.from_numpy(w_z))
    x = torch.full((B, n_buf + n_known, D), float("nan"), device="cuda")
    binding.encoder_input(x, dev[0], dev[1], w_dev, dev[2], dev[3], dev[4], B, n_buf, n_img, n_known, D, C)
    torch.cuda.synchronize()
    got = x.cpu().numpy()
    for b in range(B):
        ref = mar.encoder_input(cls[b], tok[b], w_z, b_z, pe, [n_buf + int(p) for p in known[b]], n_buf)
        e = rel_err(got[b], ref)
        assert e <= 1e-6, (b, e)
