"""Cache-aware layers split into ranges of consecutive images, each range on
its own HIP stream (marche_step_images), against the whole batch in one call.

Images are independent and every kernel computes a row (or an image and head)
the same way whatever else shares the launch -- where the number of rows picks
another kernel, that one sums in the same order -- so the KV cache and the
residual stream must match bit for bit over full and cache-aware steps, in bf16
and fp32, with the ranges overlapping on the GPU or run one after another."""
import pytest
import torch

from paper_2506_12035_amd import driver, workload
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

STEPS = range(5)  # full step 0, cache-aware 1-2, periodic full 3, cache-aware 4


@pytest.fixture(scope="module")
def whole():
    cfg = workload.CONFIGS[2]
    ws = workload.all_weights(cfg)
    eng = driver.Engine(cfg, weights=ws)
    for t in STEPS:
        eng.step(t)
    torch.cuda.synchronize()
    return cfg, ws, eng


@pytest.mark.parametrize("parts,overlap", [(2, True), (3, True), (2, False)])
def test_image_ranges_match_the_whole_batch(whole, parts, overlap):
    cfg, ws, ref = whole
    say(f"image ranges: {cfg.name} B={ref.B} parts={parts} overlap={overlap}")
    eng = driver.Engine(cfg, weights=ws, micro_batches=parts)
    eng.overlap = overlap
    assert sum(n for _, n in eng.ranges) == ref.B
    for t in STEPS:
        eng.step(t)
        if not eng.plans[t].full:
            assert eng.plans[t].parts is not None and len(eng.plans[t].parts) == parts
    torch.cuda.synchronize()
    assert torch.equal(eng.x, ref.x)
    for l in range(cfg.n_layers):
        assert torch.equal(eng.k_layer(l), ref.k_layer(l)), f"K of layer {l}"
        assert torch.equal(eng.v_layer(l), ref.v_layer(l)), f"V of layer {l}"
    for t in STEPS:
        if not eng.plans[t].full:
            assert torch.equal(eng.plans[t].ca_idx, ref.plans[t].ca_idx), f"active lists of step {t}"


@pytest.mark.timeout(600)
def test_headline_ranges_match_the_whole_batch():
    """The benchmark's default launch configuration at the headline MAR-L
    size (batch 128, 32 layers): every step as two 64-image ranges on two
    streams gives the same bits as the whole batch in one call, over full and
    cache-aware steps.  Together with the stack parity test (whole batch
    against the oracle) this covers the configuration the benchmark times."""
    cfg = workload.CONFIGS[3]
    say(f"image ranges: {cfg.name} B={cfg.batch} default ranges vs one call")
    ws = workload.all_weights(cfg)
    ref = driver.Engine(cfg, weights=ws)
    for t in STEPS:
        ref.step(t)
    torch.cuda.synchronize()
    x_ref = ref.x.clone()
    k_ref = [ref.k_layer(l).clone() for l in range(cfg.n_layers)]
    v_ref = [ref.v_layer(l).clone() for l in range(cfg.n_layers)]
    del ref
    torch.cuda.empty_cache()
    eng = driver.Engine(cfg, weights=ws, micro_batches=2)
    assert [n for _, n in eng.ranges] == [64, 64]
    for t in STEPS:
        eng.step(t)
    torch.cuda.synchronize()
    assert torch.equal(eng.x, x_ref)
    for l in range(cfg.n_layers):
        assert torch.equal(eng.k_layer(l), k_ref[l]), f"K of layer {l}"
        assert torch.equal(eng.v_layer(l), v_ref[l]), f"V of layer {l}"


def test_uneven_range_sizes_match_the_whole_batch(whole):
    """Explicit image counts per range (Engine(range_sizes=...)): unequal
    ranges, the first larger than the rest, give the same bits as one call."""
    cfg, ws, ref = whole
    sizes = [ref.B // 2 + 3, ref.B // 4, ref.B - (ref.B // 2 + 3) - ref.B // 4]
    say(f"image ranges: {cfg.name} B={ref.B} sizes={sizes}")
    eng = driver.Engine(cfg, weights=ws, range_sizes=sizes)
    assert [n for _, n in eng.ranges] == sizes
    assert [f for f, _ in eng.ranges] == [0, sizes[0], sizes[0] + sizes[1]]
    for t in STEPS:
        eng.step(t)
    torch.cuda.synchronize()
    assert torch.equal(eng.x, ref.x)
    for l in range(cfg.n_layers):
        assert torch.equal(eng.k_layer(l), ref.k_layer(l)), f"K of layer {l}"
        assert torch.equal(eng.v_layer(l), ref.v_layer(l)), f"V of layer {l}"


def test_ranges_take_tiles_for_a_shared_chip():
    """32 images in a call of their own and as one of two ranges: the ranges'
    products take the tile that leaves the other range its share of the chip."""
    from paper_2506_12035_amd import binding

    cfg = workload.CONFIGS[2].with_(n_layers=3, batch=64)
    say(f"tiles of ranges: {cfg.name} B={cfg.batch}, L=3")
    ws = workload.all_weights(cfg)
    tiles = {}
    for batch, parts in ((32, 1), (64, 2)):
        eng = driver.Engine(cfg.with_(batch=batch), weights=ws, micro_batches=parts)
        binding.profile_reset()
        binding.profile_enable(True)
        try:
            eng.step(0)
            tiles[parts] = set(binding.profile_collect())
        finally:
            binding.profile_enable(False)
            binding.profile_reset()
    assert {"gemm_o_t256x128", "gemm_fc2_t256x128"} <= tiles[1], sorted(tiles[1])
    assert {"gemm_o_t256", "gemm_fc2_t256"} <= tiles[2], sorted(tiles[2])


def test_step_images_touches_only_its_range():
    """marche_step_images on images [2, 4) of a 4-image cache and residual
    stream: images 0 and 1 keep every bit of x and of both caches, and images
    2 and 3 equal what marche_step over all four images computes for them."""
    import numpy as np
    from paper_2506_12035_amd import binding

    cfg = workload.CONFIGS[2].with_(n_layers=2, batch=4)
    B, N, D, H, dh, L = 4, cfg.n_tokens, cfg.d_model, cfg.n_heads, cfg.head_dim, 2
    say(f"marche_step_images: {cfg.name} reduced to L={L}, B={B}, images [2, 4)")
    rng = np.random.default_rng(5)
    model = binding.make_model(L, D, H, dh, cfg.d_mlp, N, binding.MARCHE_BF16, cfg.ln_eps)
    params = []
    for l in range(L):
        w = workload.layer_weights(cfg, l)
        params.append({k: torch.from_numpy(np.ascontiguousarray(v, np.float32)).to(
            torch.bfloat16 if k.startswith("w_") else torch.float32).cuda() for k, v in w.items()})
    layers = binding.make_layers(params)
    x0 = torch.from_numpy(rng.standard_normal((B, N, D)).astype(np.float32)).cuda()
    n_el = L * B * H * N * dh
    k0 = torch.from_numpy(rng.standard_normal(n_el).astype(np.float32)).to(torch.bfloat16).cuda()
    v0 = torch.from_numpy(rng.standard_normal(n_el).astype(np.float32)).to(torch.bfloat16).cuda()
    act = [np.sort(rng.choice(N, size=a, replace=False)).astype(np.int32) for a in (40, 37, 44, 29)]
    n_gen = [5, 4, 6, 3]

    def run(first, count):
        x = x0.clone()
        k, v = k0.clone(), v0.clone()
        cache = binding.kv_cache_init(model, B, k, v, n_el * 2, k_init=k0, v_init=v0)
        lists = act[first:first + count]
        idx = torch.from_numpy(np.concatenate(lists)).cuda()
        off = torch.from_numpy(np.concatenate([[0], np.cumsum([len(a) for a in lists])]).astype(np.int32)).cuda()
        gen = torch.tensor(n_gen[first:first + count], dtype=torch.int32).cuda()
        total, a_max = int(off[-1]), max(len(a) for a in lists)
        wsb = binding.workspace_bytes(model, count, total)
        ws = torch.empty(wsb, dtype=torch.uint8).cuda()
        binding.marche_step_images(model, layers, cache, first, 0, L, count, x[first:first + count],
                                   idx, off, gen, total, a_max, max(n_gen[first:first + count]),
                                   None, -1, ws, wsb)
        torch.cuda.synchronize()
        return x, k.view(L, B, H, N, dh), v.view(L, B, H, N, dh)

    x_all, k_all, v_all = run(0, 4)
    x_part, k_part, v_part = run(2, 2)
    k_in, v_in = k0.view(L, B, H, N, dh), v0.view(L, B, H, N, dh)
    assert torch.equal(x_part[:2], x0[:2])
    assert torch.equal(k_part[:, :2], k_in[:, :2]) and torch.equal(v_part[:, :2], v_in[:, :2])
    assert torch.equal(x_part[2:], x_all[2:])
    assert torch.equal(k_part[:, 2:], k_all[:, 2:]) and torch.equal(v_part[:, 2:], v_all[:, 2:])
    assert not torch.equal(x_part[2:], x0[2:])  # the range was really computed


def _layer_ranges(cfg, sizes, cuts, want_scores=True):
    """One block over images with ragged lists, in one call and as the ranges
    that `cuts` makes of the images: the same bits of x and both caches (and
    of the scores, where asked for)."""
    import numpy as np
    from tests.gpu_util import SingleLayer

    say(f"layer ranges: {cfg.name} N={cfg.n_tokens} sizes={sizes[:6]}.. cuts={cuts}")
    rng = np.random.default_rng(sum(sizes) + cfg.n_tokens)
    B, N = len(sizes), cfg.n_tokens
    x = rng.standard_normal((B, N, cfg.d_model), dtype=np.float32)
    k, v = (workload.round_to(rng.standard_normal((B, cfg.n_heads, N, cfg.head_dim), dtype=np.float32),
                              cfg.dtype) for _ in range(2))
    act = [rng.permutation(N)[:s].astype(np.int32) for s in sizes]
    gens = [min(5, s) for s in sizes]
    p = workload.layer_weights(cfg, 0)
    ref = SingleLayer(cfg, p, x, k, v).run(act, gens, want_scores)
    for a, b in zip([0] + cuts, cuts + [B]):
        got = SingleLayer(cfg, p, x[a:b], k[a:b], v[a:b]).run(act[a:b], gens[a:b], want_scores)
        for name in ("x", "k", "v") + (("scores",) if want_scores else ()):
            assert np.array_equal(got[name], ref[name][a:b]), f"{name} of images {a}..{b - 1}"
    assert not np.array_equal(ref["x"], x)


# (d_model, heads, head_dim, d_mlp, N, active rows per image, first images of the
# ranges).  Whole batches of 2560 and 1335 rows take the 64x64 tile in every
# product (K = 256, 768, 3072: slices of 16, 48 and 192), their ranges down to
# one image the kernel that splits K over wavefronts.
F32_RANGES = [
    (768, 12, 64, 3072, 320, [320] * 8, [4]),
    (768, 12, 64, 3072, 320, [320] * 8, [1]),
    (256, 4, 64, 1024, 190, [190] * 24 + [5], [2, 24]),
    (1280, 16, 80, 512, 203, [203] * 6 + [3, 41], [1, 6, 7]),
]


@pytest.mark.parametrize("case", F32_RANGES, ids=lambda c: f"d{c[0]}n{c[4]}b{len(c[5])}r{len(c[6]) + 1}")
def test_f32_ranges_match_the_whole_batch(case):
    """fp32 products take one of two kernels by their number of rows; an
    image's rows are summed in the same order by both."""
    d, h, dh, f, n, sizes, cuts = case
    cfg = workload.Config(63, "f32-ranges", 1, d, h, dh, f, n, 0, len(sizes), "f32")
    _layer_ranges(cfg, sizes, cuts)


# Whole batches of at least two (image, head) pairs per compute unit run the
# attention with all keys in LDS, smaller ranges a streaming kernel over several
# query chunks: head widths and key counts of each (N = 320 at width 64: the
# register-staged one; a key tail, heads of 80: the general one).
ATTENTION_RANGES = [
    (1024, 16, 64, 320),
    (1024, 16, 64, 289),
    (1280, 16, 80, 320),
    (1280, 16, 80, 229),
]


@pytest.mark.parametrize("case", ATTENTION_RANGES, ids=lambda c: f"h{c[2]}n{c[3]}")
def test_attention_ranges_match_the_whole_batch(case):
    from paper_2506_12035_amd import binding

    d, h, dh, n = case
    images = 2 * torch.cuda.get_device_properties(0).multi_processor_count // h + 1
    sizes = ([n, 129, 33, 200, 1] * images)[:images]
    cfg = workload.Config(65, "attn-ranges", 1, d, h, dh, 256, n, 0, images, "bf16")
    binding.profile_reset()
    binding.profile_enable(True)
    try:
        _layer_ranges(cfg, sizes, [2, 5, images // 2], want_scores=False)
        prof = binding.profile_collect()
    finally:
        binding.profile_enable(False)
        binding.profile_reset()
    assert "attention_res_ca" in prof and {"attention_q128_ca", "attention_q256_ca"} & set(prof), sorted(prof)
