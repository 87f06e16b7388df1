"""GPU parity of the many-token projection kernels, through hpd_decode_step,
against the fp64 oracle.

Token counts off the 32-token tile and off the kernels' 2- and 4-tile groups,
K of one ring up to many, hidden sizes above the prefetched sums of squares, and
a K that only the skinny kernel takes (intermediate 384).  KERNELS names the
shape that each projection takes and so keeps every kernel covered."""

import pytest
import torch

from oracle.decode import decode_step
from paper_2607_18839_amd.torch_api import DecodeStep
from workloads import get_config, make_decode_inputs

from ._gpu import BF16_MAX_ABS, BF16_REL_L2, announce, errors
from .test_gemm_choice import choose_gemm
from .test_gpu_decode import _check_cache, run_decode

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (content branches, hidden, intermediate, query heads, kv heads); 4 tokens a branch and 1 for the layout
SHAPES = [(69, 512, 1024, 16, 2),     # 277 tokens: 9 tiles
          (165, 512, 1536, 16, 8),    # 661: 21 tiles
          (250, 256, 384, 8, 2),      # 1,001: 32 tiles, one ring of K, down skinny
          (255, 1024, 3072, 16, 2),   # 1,021: 32
          (72, 2048, 1024, 8, 1)]     # 289: 10 tiles, 64 sums of squares per token
# the same, and the kernel (GemmShape.wide) of QKV, O, gate/up and down with packed and with row-major weights;
# 17, 25 and 43 tiles leave 1, 1 and 3 tiles in the last group of 4
KERNELS = [((135, 256, 2048, 8, 2), (0, 0, 2, 0), (0, 0, 4, 0)),
           ((83, 512, 4096, 8, 2), (1, 0, 4, 0), (2, 0, 4, 0)),
           ((131, 2048, 2048, 16, 2), (1, 2, 4, 2), (2, 2, 2, 2)),    # 64 sums of squares: past 4 tiles' 32
           ((197, 1024, 1024, 64, 2), (4, 1, 2, 1), (4, 2, 2, 2)),
           ((340, 2560, 1024, 8, 2), (2, 2, 4, 4), (2, 4, 2, 4))]     # 80: past 2 tiles' 64 too


def kernels(shape, packed):
    content, hidden, inter, hq, hkv = shape
    tiles = (4 * content + 1 + 31) // 32
    sizes = (("qkv", (hq + 2 * hkv) * 64, hidden), ("o", hidden, hq * 64), ("gate_up", 2 * inter, hidden),
             ("down", hidden, inter))
    return tuple(choose_gemm(use, n, k, tiles, packed)[1] for use, n, k in sizes)


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "torch"])
@pytest.mark.parametrize("case", KERNELS, ids=lambda c: "-".join(map(str, c[0])))
def test_every_kernel(case, packed):
    shape, want_packed, want_torch = case
    assert kernels(shape, packed) == (want_packed if packed else want_torch)
    test_many_tokens(shape, packed)


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "torch"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_many_tokens(shape, packed):
    content, hidden, inter, hq, hkv = shape
    announce(f"decode many tokens {shape} packed {packed}")
    cfg = get_config("c4", num_q_heads=hq, num_kv_heads=hkv, num_pages=1, prefix=("fixed", 70),
                     layout=dict(k=1, past=("fixed", 5)), content_count=("fixed", content), content_k=4,
                     content_past=("lognormal", 4.0, 1.0, 0, 20),
                     model=dict(num_layers=2, hidden=hidden, intermediate=inter, weight_std=0.02, rms_eps=1e-6))
    inp = make_decode_inputs(cfg, 3)
    h, pk, pv = run_decode(inp, packed=packed)
    ref, nk, nv = decode_step(inp)
    mx, rl = errors(h, ref)
    print(f"{shape} packed {packed}: max abs {mx:.3e} rel L2 {rl:.3e}")
    assert mx <= BF16_MAX_ABS and rl <= BF16_REL_L2, (mx, rl)
    _check_cache(inp, pk, pv, nk, nv)


@pytest.mark.parametrize("shape", [(69, 512, 1024), (340, 512, 1536), (83, 512, 4096)],
                         ids=lambda s: "-".join(map(str, s)))
def test_swiglu_is_the_same_in_every_kernel(shape):
    """Hidden values that are powers of two and one weight per gate, up and down
    row: every product and sum is exact, so that the packed kernels of 1, 2 and
    4 token tiles and the row-major ones can differ in SwiGLU itself alone."""
    content, hidden, inter = shape
    announce(f"swiglu {shape}")
    T, g = 4 * content + 1, torch.Generator().manual_seed(content)
    wide = kernels((content, hidden, inter, 8, 2), True)[2]
    assert wide == {69: 1, 340: 2, 83: 4}[content]

    def one_per_row(rows, cols, values):
        w = torch.zeros(rows, cols)
        w[torch.arange(rows), torch.randint(cols, (rows,), generator=g)] = values
        return w.bfloat16().cuda()

    weights = dict(w_qkv=torch.randn(12 * 64, hidden, generator=g).bfloat16().cuda(),
                   w_o=torch.zeros(hidden, 512).bfloat16().cuda(),
                   w_gate=one_per_row(inter, hidden, 2 * torch.randn(inter, generator=g)),
                   w_up=one_per_row(inter, hidden, torch.randn(inter, generator=g)),
                   w_down=one_per_row(hidden, inter, torch.ones(hidden)))
    h = torch.randint(-2, 2, (T, hidden), generator=g).float().exp2()
    h *= torch.randint(2, (T, hidden), generator=g) * 2 - 1
    out = []
    for packed in (True, False):
        step = DecodeStep(8, 2, [64], [0] * (content + 1), [1] + [4] * content, [0] * (content + 1),
                          {n: [w] for n, w in weights.items()}, hidden, inter, packed=packed)
        kv = [[torch.zeros(n, 2, 64, dtype=torch.bfloat16, device="cuda")] for n in (64, 64, T, T)]
        out.append(step(h.cuda(), *kv))
    m = out[0] - h.cuda()
    assert torch.isfinite(m).all() and (m != 0).float().mean() > 0.9
    assert torch.equal(out[0], out[1]), int((out[0] != out[1]).sum())
