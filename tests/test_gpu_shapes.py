"""One block at the edges of the launch rules, against the fp64 oracle: fp32
products of one row, of 16 / 32 / 64-row remainders and of enough rows for the
64x64 tile; fp32 attention with one and with four rows per workgroup; bf16
attention on ragged key tails at both head widths, with few (image, head)
pairs (two key groups per workgroup) and with many, for one to four query
blocks, with the score pass as a kernel of its own."""
import numpy as np
import pytest

from paper_2506_12035_amd import workload
from tests.gpu_util import TOL, SingleLayer, f64, say
from tests.test_gpu_layer import _check_layer, _oracle_layer

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


# Two images: at most 32 (image, head) pairs per query block; nine images: 144
# and more.  Lists up to 32, 64, 128 and more rows; key tails of 1 and 37 (an
# aligned length too: it takes the streaming kernel of its own with many
# pairs).  More than 64 generating rows need the separate score pass at every
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
