"""Dispatch and combine of few tokens, around the row count where dispatch takes another form."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from harness import f64
from paper_2602_21140_amd import ReviveLayer

pytestmark = pytest.mark.gpu


# (T, k, P, H): one row, ragged last words of a row, 1023 to 1026 routed rows, the most slots and choices
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("T,k,P,H", [(0, 2, 20, 64), (1, 1, 1, 64), (1, 8, 288, 7168), (37, 6, 72, 2112), (341, 3, 1023, 128), (32, 32, 1024, 448),
                                     (512, 2, 1024, 64), (511, 2, 40, 2048), (513, 2, 256, 320), (1024, 1, 7, 64), (1025, 1, 900, 64)])
def test_dispatch_and_combine(T, k, P, H, static):
    rng = np.random.default_rng(T + P)
    E = max(k, min(P, 512))
    cfg = SimpleNamespace(T=max(T, 1), H=H, E=E, k=k, I=64, I_shared=0, n_ranks=1, slots_per_rank=P, max_replicas=4,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="bf16")
    L = ReviveLayer(cfg)
    slots = rng.integers(0, P, size=T * k).astype(np.int32)
    if T > 1:  # ids that name no slot: those rows are dropped
        slots[rng.integers(0, T * k, size=3)] = [-1, P, 2 ** 31 - 1]
    valid = (slots >= 0) & (slots < P)
    order = np.argsort(np.where(valid, slots, P), kind="stable")[:valid.sum()]
    dst = np.full(T * k, -1, dtype=np.int32)
    dst[order] = np.arange(len(order))
    off = np.concatenate([[0], np.cumsum(np.bincount(slots[valid], minlength=P))])
    x = torch.randn(max(T, 1), H, device="cuda").to(torch.bfloat16)
    tp = torch.from_numpy(slots).cuda()
    n = max(1, T * k)
    out = (torch.full((n, H), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.full((P + 1,), -7, dtype=torch.int32, device="cuda"),
           torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.full((n,), -7, dtype=torch.int32, device="cuda"))
    for _ in range(2):
        xp, offs, dr, so = L.dispatch(x, tp, T, out=out, static_scratch=static)
    assert np.array_equal(offs.cpu().numpy(), off)
    assert np.array_equal(dr.cpu().numpy()[:T * k], dst)
    assert np.array_equal(so.cpu().numpy()[:len(order)], order)
    assert torch.equal(xp[:len(order)], x[torch.from_numpy(order // k).cuda()])
    if T:
        w = torch.rand(T, k, device="cuda")
        y = torch.where(torch.arange(n, device="cuda")[:, None] < len(order), xp, torch.zeros_like(xp))
        got = L.combine(y, dr, w, None, T)
        rows = np.where(dst[:, None] >= 0, f64(y)[np.maximum(dst, 0)], 0.0).reshape(T, k, H)
        ref = (f64(w)[:, :, None] * rows).sum(axis=1)
        # one rounding to bf16 (2^-9 of the value) after an fp32 sum of at most 32 terms
        assert (np.abs(f64(got) - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5).all()
    L.close()
