"""Router logits at the token and expert counts where a tile, a K step or a rule of the launch ends, against
fp64 products of the same bits."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2602_21140_amd import ReviveLayer

pytestmark = pytest.mark.gpu


# (T, E, H): 16 x 16 tiles (one token to several tiles, ragged in both), 32 x 32 tiles from 256 workgroups on, seven
# and eight token tiles, fewer steps of K than wavefronts, the GEMM's tiles of 64 and of 128 experts, K in slices there
SHAPES = [(1, 16, 64), (15, 24, 192), (17, 16, 448), (112, 40, 512), (113, 40, 576), (129, 256, 704), (1000, 256, 320),
          (1025, 250, 448), (4090, 256, 128), (4100, 130, 1024), (65500, 70, 64), (32700, 200, 128), (16400, 128, 1024),
          (65601, 128, 256)]
F32_H = {64: 8, 192: 40, 448: 1000, 320: 72}


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,E,H", SHAPES)
def test_router_logits(T, E, H, dtype):
    if dtype == "fp32":
        H = F32_H.get(H, H)
    cfg = SimpleNamespace(T=T, H=H, E=E, k=1, I=64, I_shared=0, n_ranks=1, slots_per_rank=E, max_replicas=1,
                          score_fn="softmax", n_group=1, topk_group=1, dtype=dtype)
    L = ReviveLayer(cfg)
    L.set_placement(np.arange(E, dtype=np.int32))
    L.update_map(np.zeros(1, dtype=np.uint8))
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(T, H, generator=gen, device="cuda").to(L.dtype)
    w = (torch.randn(E, H, generator=gen, device="cuda") * H ** -0.5).to(L.dtype)
    logits = torch.full((T, E), float("nan"), device="cuda")
    L.route(x, w, T, logits=logits)
    again = torch.full((T, E), float("nan"), device="cuda")
    L.route(x, w, T, logits=again)
    exact = x.double() @ w.double().T
    # exact products; a sum of H <= 1024 rounds H times to 2^-24 of a partial sum: below 2^-24 sqrt(1024) = 2e-6
    # of the logit's standard deviation (1), less where the sum is split
    assert (logits.double() - exact).abs().max().item() < 2e-5  # ten times that for the largest of 10^7
    assert ((logits.double() - exact).norm() / exact.norm()).item() < 2e-6
    assert torch.equal(logits, again)
    L.close()


# a token's logits do not depend on the other tokens of the call: one, a few, as many as change the kernel
@pytest.mark.parametrize("dtype,E,H", [("bf16", 256, 7168), ("bf16", 200, 448), ("bf16", 40, 576), ("bf16", 64, 2048),
                                       ("bf16", 128, 7168), ("bf16", 128, 256), ("fp32", 64, 1000),
                                       ("fp32", 256, 392), ("fp32", 512, 40)])
def test_logits_do_not_depend_on_the_token_count(dtype, E, H):
    n = 66000 if H == 256 else 9000  # with 128 experts more than 2336 tokens at H = 7168, 65536 at 256, are the GEMM's
    cfg = SimpleNamespace(T=n, H=H, E=E, k=1, I=64, I_shared=0, n_ranks=1, slots_per_rank=E, max_replicas=1,
                          score_fn="softmax", n_group=1, topk_group=1, dtype=dtype)
    L = ReviveLayer(cfg)
    L.set_placement(np.arange(E, dtype=np.int32))
    L.update_map(np.zeros(1, dtype=np.uint8))
    gen = torch.Generator(device="cuda").manual_seed(E)
    x = torch.randn(n, H, generator=gen, device="cuda").to(L.dtype)
    w = (torch.randn(E, H, generator=gen, device="cuda") * H ** -0.5).to(L.dtype)
    whole = L.route(x, w, n)[0]
    for T in (1, 17, 500, 512, 513, 2336, 2337, 4100):
        assert torch.equal(L.route(x[:T].contiguous(), w, T)[0], whole[:T]), T
    L.close()


# K in one sequence: every tile size of the router (the limits are those of E = 256), a K that does not fill the last step
# of 128 elements, one shorter than it, ragged experts; 192 and 256 experts per column tile
@pytest.mark.parametrize("E,H", [(256, 192), (300, 448), (130, 128), (200, 64), (384, 320)])
def test_every_tile_gives_the_same_bits(E, H):
    n = 33000
    cfg = SimpleNamespace(T=n, H=H, E=E, k=1, I=64, I_shared=0, n_ranks=1, slots_per_rank=E, max_replicas=1,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="bf16")
    L = ReviveLayer(cfg)
    L.set_placement(np.arange(E, dtype=np.int32))
    L.update_map(np.zeros(1, dtype=np.uint8))
    gen = torch.Generator(device="cuda").manual_seed(E)
    x = torch.randn(n, H, generator=gen, device="cuda").to(L.dtype)
    w = (torch.randn(E, H, generator=gen, device="cuda") * H ** -0.5).to(L.dtype)
    whole = L.route(x, w, n)[0]
    exact = x.double() @ w.double().T
    assert (whole.double() - exact).abs().max().item() < 2e-5  # as in test_router_logits
    for T in (1, 8, 9, 64, 65, 256, 257, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16000, 32640, 32641):
        logits = torch.full((T, E), float("nan"), device="cuda")
        assert torch.equal(L.route(x[:T].contiguous(), w, T, logits=logits)[0], whole[:T]), T
    L.close()


# few experts, which take narrow tiles with many tokens, and experts of which one round of 128 x 128 tiles just does not do
@pytest.mark.parametrize("E,H", [(40, 704), (100, 576), (16, 64), (130, 64)])
def test_every_tile_gives_the_same_bits_few_experts(E, H):
    test_every_tile_gives_the_same_bits(E, H)


# few experts, K in slices: past one round of narrow tiles, of wide ones, and far past both
@pytest.mark.parametrize("T,E", [(32769, 40), (16385, 100), (32769, 70), (49200, 128)])
def test_router_logits_in_slices(T, E):
    test_router_logits(T, E, 1024, "bf16")
