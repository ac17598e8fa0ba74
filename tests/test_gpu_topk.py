"""Selection on given logits at the expert, group and token counts where the kernel takes another form, with
many equal logits, against the oracle."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from harness import f64
from oracle import revive_oracle as orc
from paper_2602_21140_amd import ReviveLayer

pytestmark = pytest.mark.gpu

# E, n_group, topk_group, k: groups that are aligned runs of 8, 16, 32 and 64 lanes, groups that are not (24, 48, 25,
# 128, 4 experts), more groups than the four-token form takes, more choices than it takes, no groups
SHAPES = [(64, 8, 3, 6), (128, 8, 4, 8), (256, 8, 4, 8), (512, 8, 4, 8), (192, 8, 4, 5), (384, 8, 2, 3), (200, 8, 2, 16),
          (256, 2, 1, 8), (32, 8, 8, 16), (512, 32, 8, 32), (320, 20, 3, 8), (256, 8, 4, 17), (61, 1, 1, 1), (384, 1, 1, 8), (500, 1, 1, 32)]


@pytest.mark.parametrize("T", [1, 301, 8193])
@pytest.mark.parametrize("score_fn", ["softmax", "sigmoid"])
@pytest.mark.parametrize("E,n_group,topk_group,k", SHAPES)
def test_topk(E, n_group, topk_group, k, score_fn, T):
    rng = np.random.default_rng(E + k)
    slots = -(-E * 5 // 4)
    p2l = np.concatenate([np.arange(E), rng.permutation(E)[:slots - E]]).astype(np.int32)  # some experts twice
    cfg = SimpleNamespace(T=T, H=64, E=E, k=k, I=64, I_shared=0, n_ranks=1, slots_per_rank=slots, max_replicas=2,
                          score_fn=score_fn, n_group=n_group, topk_group=topk_group, dtype="bf16")
    L = ReviveLayer(cfg)
    L.set_placement(p2l)
    lost = np.zeros(E, dtype=np.uint8)
    lost[rng.permutation(E)[:E // 16]] = 1
    L.update_map(np.zeros(1, dtype=np.uint8), expert_failed=lost)
    logits = torch.from_numpy(np.round(rng.standard_normal((T, E)) * 8) / 8).float().cuda()  # eighths: many ties
    _, top, w, phys = L.route(None, None, T, logits=logits, logits_given=True)
    m = orc.build_map(p2l, np.zeros(1, dtype=np.uint8), slots, E, 2, expert_failed=lost)
    s = orc.scores(f64(logits), score_fn)
    ref = orc.select_topk(orc.masked_selection_scores(s, m.l2p_count), k, n_group, topk_group)
    assert np.array_equal(top.cpu().numpy(), ref)
    assert np.array_equal(phys.cpu().numpy(), orc.remap(ref, m))
    assert np.abs(f64(w) - orc.gate_weights(s, ref)).max() < 2e-7  # one rounding to fp32 of a weight below 1
    L.close()


# 16 lanes per token: as many experts per lane as a form of the kernel holds, one more and fewer, experts that are no
# multiple of 4 or of 16, groups of 2, 4 and 8 lanes, one choice and sixteen; both sides of the limits in tokens
@pytest.mark.parametrize("T", [16, 17, 19, 2048, 2049])
@pytest.mark.parametrize("E,n_group,topk_group,k", [(2, 1, 1, 1), (30, 1, 1, 16), (80, 1, 1, 4), (112, 1, 1, 8), (144, 1, 1, 8), (192, 1, 1, 6),
                                                    (48, 2, 1, 8), (48, 4, 2, 3), (48, 8, 3, 2), (128, 4, 1, 16), (208, 2, 1, 16),
                                                    (256, 8, 4, 8), (320, 4, 3, 7), (400, 1, 1, 2), (512, 2, 2, 16), (511, 1, 1, 5)])
def test_a_row_of_lanes_per_token(E, n_group, topk_group, k, T):
    test_topk(E, n_group, topk_group, k, "sigmoid" if k % 2 else "softmax", T)


# the same from the token counts on at which layers without groups, and wide ones with few lanes per load, take this kernel
@pytest.mark.parametrize("T", [2560, 4099])
@pytest.mark.parametrize("E,n_group,topk_group,k", [(2, 1, 1, 1), (30, 1, 1, 16), (80, 1, 1, 4), (112, 1, 1, 8), (130, 1, 1, 2), (144, 1, 1, 8),
                                                    (192, 1, 1, 6), (300, 1, 1, 8), (400, 2, 1, 8), (448, 1, 1, 16), (500, 1, 1, 1),
                                                    (511, 1, 1, 5), (512, 1, 1, 1), (512, 2, 2, 16)])
def test_a_row_of_lanes_per_token_many_tokens(E, n_group, topk_group, k, T):
    test_topk(E, n_group, topk_group, k, "softmax" if k % 2 else "sigmoid", T)


# four tokens to a wavefront, the last wavefront with one: every count of logits per lane, groups that are aligned runs of
# 8, 32 and 64 lanes and groups that are not; and one token to a wavefront just before
@pytest.mark.parametrize("T", [16384, 16385])
@pytest.mark.parametrize("E,n_group,topk_group,k", [(24, 3, 2, 4), (72, 8, 3, 6), (96, 3, 1, 16), (120, 5, 2, 6), (192, 3, 2, 9), (200, 8, 2, 16),
                                                    (360, 5, 3, 8), (504, 7, 3, 16)])
def test_four_tokens_to_a_wavefront(E, n_group, topk_group, k, T):
    test_topk(E, n_group, topk_group, k, "sigmoid" if E % 3 else "softmax", T)


@pytest.mark.parametrize("E,n_group,topk_group,k", [(24, 3, 2, 4), (200, 8, 2, 16), (504, 7, 3, 8)])
def test_four_tokens_to_a_wavefront_nan(E, n_group, topk_group, k):
    test_nan_logits_are_absent_from_their_group(E, n_group, topk_group, k, "softmax", 16385)
    test_row_of_nan_keeps_valid_ids(E, n_group, k, 16385)


# places of a lane that hold no expert are never chosen, not even where all the token's logits are NaN
@pytest.mark.parametrize("E,n_group,k", [(48, 1, 8), (48, 2, 8), (400, 4, 16), (500, 1, 8), (511, 1, 16)])
def test_row_of_nan_with_a_row_of_lanes(E, n_group, k):
    test_row_of_nan_keeps_valid_ids(E, n_group, k, 8193)


# A logit that is not a number belongs to no order: its expert counts as absent, in the scores of its group too.
@pytest.mark.parametrize("T", [301, 8193])
@pytest.mark.parametrize("score_fn", ["softmax", "sigmoid"])
@pytest.mark.parametrize("E,n_group,topk_group,k", [(64, 8, 3, 6), (256, 8, 4, 8), (512, 8, 4, 8), (200, 8, 2, 16), (256, 2, 1, 8), (512, 32, 8, 32)])
def test_nan_logits_are_absent_from_their_group(E, n_group, topk_group, k, score_fn, T):
    rng = np.random.default_rng(E + n_group)
    cfg = SimpleNamespace(T=T, H=64, E=E, k=k, I=64, I_shared=0, n_ranks=1, slots_per_rank=E, max_replicas=1,
                          score_fn=score_fn, n_group=n_group, topk_group=topk_group, dtype="bf16")
    L = ReviveLayer(cfg)
    L.set_placement(np.arange(E, dtype=np.int32))
    L.update_map(np.zeros(1, dtype=np.uint8))
    z = rng.standard_normal((T, E)).astype(np.float32)
    gsz = E // n_group
    for g in range(n_group):  # beside each group's best: the neighbour that a reduction meets it with first
        best = z[:, g * gsz:(g + 1) * gsz].argmax(axis=1)
        t = np.arange(T)
        for d in (best ^ 1, (best + 64) % gsz):
            on = (d < gsz) & (d != best) & (t % 3 > 0)
            z[t[on], g * gsz + d[on]] = np.nan
    _, top, w, _ = L.route(None, None, T, logits=torch.from_numpy(z).cuda(), logits_given=True)
    s = orc.scores(np.where(np.isnan(z), -np.inf, z.astype(np.float64)), score_fn)
    ref = orc.select_topk(np.where(np.isnan(z), -np.inf, s), k, n_group, topk_group)
    assert np.array_equal(top.cpu().numpy(), ref)
    assert np.abs(f64(w) - orc.gate_weights(s, ref)).max() < 2e-7  # as above
    L.close()


# A row of nothing but NaN has no best expert: its weights are NaN, its ids and slots stay those of experts, and the
# other rows do not notice.
@pytest.mark.parametrize("T", [5, 8193])
@pytest.mark.parametrize("E,n_group,k", [(61, 1, 3), (64, 1, 3), (200, 8, 16), (200, 1, 32), (500, 4, 8)])
def test_row_of_nan_keeps_valid_ids(E, n_group, k, T):
    cfg = SimpleNamespace(T=T, H=64, E=E, k=k, I=64, I_shared=0, n_ranks=1, slots_per_rank=E, max_replicas=1,
                          score_fn="softmax", n_group=n_group, topk_group=n_group, dtype="bf16")
    L = ReviveLayer(cfg)
    L.set_placement(np.arange(E, dtype=np.int32)[::-1].copy())  # expert e in slot E - 1 - e
    L.update_map(np.zeros(1, dtype=np.uint8))
    logits = torch.randn(T, E, generator=torch.Generator().manual_seed(E)).cuda()
    _, top, w, phys = (t.cpu().numpy() for t in L.route(None, None, T, logits=logits, logits_given=True))
    bad = np.arange(T) % 4 == 2
    logits[torch.from_numpy(bad).cuda()] = float("nan")
    _, top2, w2, phys2 = (t.cpu().numpy() for t in L.route(None, None, T, logits=logits, logits_given=True))
    for a, b in ((top, top2), (w, w2), (phys, phys2)):
        assert np.array_equal(a[~bad], b[~bad])
    assert np.isnan(w2[bad]).all()
    assert (top2[bad] >= 0).all() and (top2[bad] < E).all()
    assert np.array_equal(phys2, E - 1 - top2)
    L.close()


# What NaN leave of a row is chosen alike by every kernel: a row that keeps fewer experts than it chooses, or none, takes the
# same ones in a call of many tokens and in one of few.
@pytest.mark.parametrize("T", [96, 8193, 16400])
@pytest.mark.parametrize("E,n_group,topk_group,k", [(16, 1, 1, 2), (61, 1, 1, 3), (64, 8, 4, 8), (256, 2, 2, 16), (384, 8, 8, 3), (500, 1, 1, 8), (512, 1, 1, 16), (120, 5, 2, 2)])
def test_rows_of_nan_do_not_depend_on_the_token_count(E, n_group, topk_group, k, T):
    cfg = SimpleNamespace(T=T, H=64, E=E, k=k, I=64, I_shared=0, n_ranks=1, slots_per_rank=E, max_replicas=1,
                          score_fn="sigmoid", n_group=n_group, topk_group=topk_group, dtype="bf16")
    L = ReviveLayer(cfg)
    L.set_placement(np.arange(E, dtype=np.int32))
    L.update_map(np.zeros(1, dtype=np.uint8))
    gen = torch.Generator().manual_seed(E + k)
    z = torch.randn(T, E, generator=gen)
    kind = torch.arange(T) % 4
    z[kind == 1] = float("nan")
    z[(torch.rand(T, E, generator=gen) < 0.3) & (kind == 2)[:, None]] = float("nan")
    few = kind == 3  # fewer than k left, of one group
    keep = torch.randint(0, E // n_group, (T,), generator=gen)
    left = z[torch.arange(T), keep].clone()
    z[few] = float("nan")
    z[torch.arange(T)[few], keep[few]] = left[few]
    z = z.cuda()
    _, *many = L.route(None, None, T, logits=z, logits_given=True)
    for t0 in (0, (T - 12) // 2 & ~3, T - 12):
        _, *some = L.route(None, None, 12, logits=z[t0:t0 + 12].contiguous(), logits_given=True)
        for a, b in zip(many, some):  # a weight's NaN has no sign that would say anything
            assert torch.equal(a[t0:t0 + 12].nan_to_num(nan=-1.0), b.nan_to_num(nan=-1.0)), t0
    L.close()
