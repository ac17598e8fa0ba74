"""Expert FFN with few rows per slot and in fp32, at the row counts where a row-tile ends, against plain torch."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from harness import TOL, f64, rel_err
from paper_2602_21140_amd import ReviveLayer
from paper_2602_21140_amd.binding import pack_expert

pytestmark = pytest.mark.gpu

EDGES = [1, 0, 16, 15, 17, 32, 33, 64, 0, 65, 2, 127, 128, 129, 256, 257, 300, 0]
TALL = [257, 0, 288, 289, 319, 320, 321, 256, 577, 304, 272]  # 128 rows per slot or more on average
SUB_TILES = [16 * i + d for i in range(20) for d in (1, 16)] + [321, 513, 767, 1025, 1300]
# (H, I, rows of the slots): one group of K up to several, K no multiple of the ring, columns that are half a tile
CASES = {
    "edges": (256, 192, EDGES + [0] * 90),  # up to 16 rows per slot on average the weights are always streamed
    "short_k": (64, 64, EDGES + [0] * 90),
    "odd_k": (704, 320, EDGES + [3] * 100),
    "tiles": (704, 320, EDGES + [3] * 10),  # above, at this size, the 256-row tiles
    # one row-tile up to 320 rows, from the shortest K to several turns of the ring
    "tall": (256, 192, TALL), "tall_short_k": (64, 64, TALL), "tall_long_k": (1088, 448, TALL),
    # few workgroups and cached weights: row-tiles of 64 also beside many rows of the shared expert
    "small_tiles": (704, 320, [130, 65, 64, 1, 0, 16, 3] + [0] * 13),
    # the same with enough workgroups for tall tiles
    "tall_many_short_k": (64, 64, TALL * 12), "tall_many": (192, 320, TALL * 12), "tall_wide": (2880, 1472, TALL),
    # every number of 16-row sub-tiles that a wavefront may have, full and by one row, and slots of several row-tiles
    "sub_tiles": (256, 192, SUB_TILES), "sub_tiles_tall": (1088, 448, SUB_TILES),
    # slots of many row-tiles, which a common height would leave with a row or a sub-tile in the last; the same streamed
    "many_tiles": (256, 192, [4097, 3601, 513, 0, 1]), "many_tiles_streamed": (704, 320, [4097, 1041] + [0] * 330),
    # half the columns up to 1024 workgroups, tiles of 64 rows above 8 rows per slot, of 128 above 20 (12 where they are many),
    # and for many rows of the shared expert; narrow experts, with few workgroups and cached weights and with many
    "half_columns": (1024, 1024, [1, 0, 63, 64, 65] + [2] * 32), "tiles_of_64": (2048, 576, [129, 64, 65, 1, 17] + [9] * 25),
    "tiles_of_64_wide": (2368, 576, [129, 64, 65, 1, 17] + [9] * 52), "tiles_of_128": (2048, 576, [129, 128, 127, 257, 1] + [17] * 25),
    "tiles_of_128_many": (1344, 960, [129, 128, 127, 257, 1] + [8] * 91),
    "rows_shared": (1024, 1024, [300, 100, 65, 20] + [1] * 35),
    "small_tiles_narrow": (704, 256, [130, 65, 64, 1, 0, 16, 3] + [0] * 13), "tiles_of_128_narrow": (1024, 128, [129, 128, 257, 1] + [6] * 188),
    "one_row": (448, 128, [0] * 7 + [1] + [0] * 56),
    "few": (256, 320, [5, 1, 0, 8, 3, 16, 2, 7] * 8),
    "many_slots": (128, 64, ([0, 2, 1, 65] + [0] * 12) * 60),
    "many_slots_streamed": (128, 64, ([0, 2, 1, 65] + [0] * 12) * 40),
}


def _reference(x, w):
    g, u, d = (t.float().cpu() for t in w)
    h = (torch.nn.functional.silu(x @ g) * (x @ u)).to(torch.bfloat16).float()
    return h @ d


@pytest.mark.parametrize("shared", [0, 1, 2])  # 0: none, 1: in the same call, 2: alone
@pytest.mark.parametrize("name", list(CASES))
def test_few_rows_per_slot(name, shared):
    H, I, counts = CASES[name]
    P, N = len(counts), sum(counts)
    T = N if shared < 2 else min(N, 100)
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(torch.bfloat16)

    cfg = SimpleNamespace(T=N, H=H, E=min(P, 512), k=1, I=I, I_shared=I if shared else 0, n_ranks=P, slots_per_rank=1, max_replicas=2,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="bf16")
    L = ReviveLayer(cfg)
    experts = [(normal(H, I, std=H ** -0.5), normal(H, I, std=H ** -0.5), normal(I, H, std=I ** -0.5)) if c else None for c in counts]
    packed = [pack_expert(*w) if w else (None, None) for w in experts]
    L.set_expert_weights([p[0] for p in packed], [p[1] for p in packed])
    w_sh = (normal(H, I, std=H ** -0.5), normal(H, I, std=H ** -0.5), normal(I, H, std=I ** -0.5))
    gu, dn = pack_expert(*w_sh)
    x = normal(N, H)
    y, y_sh = L.empty(N, H).fill_(float("nan")), L.empty(T, H).fill_(float("nan"))
    off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    if shared == 2:
        L.shared_ffn(x[:T].contiguous(), gu, dn, T, out=y_sh)
    else:
        L.expert_ffn(x, off, N, x=x, w_sh_gate_up=gu if shared else None, w_sh_down=dn if shared else None, out=(y, y_sh))
    torch.cuda.synchronize()
    xf = x.float().cpu()
    if shared < 2:
        for p, c in enumerate(counts):
            if c:
                a, b = int(off[p]), int(off[p + 1])
                assert rel_err(f64(y[a:b]), _reference(xf[a:b], experts[p]).double().numpy()) < TOL["bf16"], (p, c)
    if shared:
        assert rel_err(f64(y_sh), _reference(xf[:T], w_sh).double().numpy()) < TOL["bf16"]
    L.close()


# (H, I): K a multiple of the 32-wide step and not, shorter than one step, more steps than are in flight, ragged columns
@pytest.mark.parametrize("H,I", [(8, 4), (40, 36), (72, 132), (256, 128), (1000, 68)])
@pytest.mark.parametrize("shared", [0, 1, 2])
def test_fp32_row_tiles(H, I, shared):
    counts = [1, 0, 16, 15, 17, 32, 33, 48, 49, 64, 0, 65, 2, 127, 128, 129, 300, 0]
    P, N = len(counts), sum(counts)
    gen = torch.Generator(device="cuda").manual_seed(6)

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=gen, device="cuda") * std

    cfg = SimpleNamespace(T=N, H=H, E=P, k=1, I=I, I_shared=I if shared else 0, n_ranks=P, slots_per_rank=1, max_replicas=1,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="fp32")
    L = ReviveLayer(cfg)
    experts = [(normal(H, I, std=H ** -0.5), normal(H, I, std=H ** -0.5), normal(I, H, std=I ** -0.5)) if c else None for c in counts]
    packed = [pack_expert(*w) if w else (None, None) for w in experts]
    L.set_expert_weights([p[0] for p in packed], [p[1] for p in packed])
    w_sh = (normal(H, I, std=H ** -0.5), normal(H, I, std=H ** -0.5), normal(I, H, std=I ** -0.5))
    gu, dn = pack_expert(*w_sh)
    x = normal(N, H)
    y, y_sh = L.empty(N, H).fill_(float("nan")), L.empty(N, H).fill_(float("nan"))
    off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    if shared == 2:
        L.shared_ffn(x, gu, dn, N, out=y_sh)
    else:
        L.expert_ffn(x, off, N, x=x, w_sh_gate_up=gu if shared else None, w_sh_down=dn if shared else None, out=(y, y_sh))
    torch.cuda.synchronize()

    def reference(rows, w):
        g, u, d = (f64(t) for t in w)
        z = rows @ g
        return (z / (1.0 + np.exp(-z)) * (rows @ u)) @ d

    xd = f64(x)
    if shared < 2:
        for p, c in enumerate(counts):
            if c:
                a, b = int(off[p]), int(off[p + 1])
                # sums of up to a thousand fp32 products: 2^-24 sqrt(1000) = 2e-6 of the largest, five times that allowed
                assert rel_err(f64(y[a:b]), reference(xd[a:b], experts[p])) < 1e-5, (p, c)
    if shared:
        assert rel_err(f64(y_sh), reference(xd, w_sh)) < 1e-5
    L.close()


# A workgroup finds its row-tile among the slots by itself: a lane adds up ceil(P / 64) of them.
@pytest.mark.parametrize("P", [1, 2, 63, 64, 65, 127, 128, 129, 320, 321, 961, 1024])
def test_row_tiles_among_the_slots(P):
    H, I = 16, 8
    rng = np.random.default_rng(P)
    for fill in (0.05, 0.5, 1.0):  # share of the slots that have rows, in one to three row-tiles
        counts = np.where(rng.random(P) < fill, rng.integers(1, 150 if P < 100 else 8, P), 0)
        counts[rng.integers(P)] = 130
        N = int(counts.sum())
        cfg = SimpleNamespace(T=N, H=H, E=min(P, 512), k=1, I=I, I_shared=0, n_ranks=P, slots_per_rank=1, max_replicas=2,
                              score_fn="softmax", n_group=1, topk_group=1, dtype="fp32")
        L = ReviveLayer(cfg)
        gen = torch.Generator(device="cuda").manual_seed(P)
        gu, dn = torch.randn(P, 2 * I, H, generator=gen, device="cuda"), torch.randn(P, H, I, generator=gen, device="cuda")
        L.set_expert_weights([gu[p] if c else None for p, c in enumerate(counts)], [dn[p] if c else None for p, c in enumerate(counts)])
        x, y = torch.randn(N, H, generator=gen, device="cuda"), L.empty(N, H).fill_(float("nan"))
        off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
        L.expert_ffn(x, off, N, out=(y, None))
        slot = torch.from_numpy(np.repeat(np.arange(P), counts)).cuda()
        z = (gu[slot].double() * x.double()[:, None, :]).sum(2)
        ref = (dn[slot].double() * (torch.nn.functional.silu(z[:, :I]) * z[:, I:])[:, None, :]).sum(2)
        assert float((y - ref).abs().max() / ref.abs().max()) < 1e-5, fill  # sums of at most 16 fp32 products
        L.close()


# fp32 on the bf16 matrix cores, at every number of 16-row sub-tiles and K-steps from one up, even and odd, full and not.
# Rows and weights whose bf16 parts are no numbers (the largest fp32 values, infinities, NaN) go through sums in fp32; the
# other rows of their tiles keep their bits.
@pytest.mark.parametrize("H,I", [(16, 8), (32, 36), (40, 64), (96, 100), (1024, 512)])
@pytest.mark.parametrize("rows", [1, 16, 17, 33, 64, 65])
def test_fp32_parts_and_numbers_without_parts(H, I, rows):
    gen = torch.Generator(device="cuda").manual_seed(10)
    cfg = SimpleNamespace(T=2 * rows, H=H, E=2, k=1, I=I, I_shared=0, n_ranks=2, slots_per_rank=1, max_replicas=1,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="fp32")
    L = ReviveLayer(cfg)
    g, u, d = (torch.randn(*s, generator=gen, device="cuda") * s[0] ** -0.5 for s in ((H, I), (H, I), (I, H)))
    g[5] *= 2e-38
    u[5] *= 2e-38
    gu, dn = pack_expert(g, u, d)
    L.set_expert_weights([gu, gu], [dn, dn])
    x = torch.randn(2 * rows, H, generator=gen, device="cuda")
    off = torch.tensor([0, rows, 2 * rows], dtype=torch.int32, device="cuda")

    def run():
        y = L.empty(2 * rows, H).fill_(-7.0)
        L.expert_ffn(x, off, 2 * rows, out=(y, None))
        torch.cuda.synchronize()
        return y

    def reference():
        z, w = x.double() @ g.double(), x.double() @ u.double()
        return (torch.nn.functional.silu(z) * w) @ d.double()

    plain, ref = run(), reference()
    # a K-step rounds the leading sum once, by 2^-24 of it at most, in one direction or the other; h and y are rounded once
    # more.  Measured: 0.6e-7 to 3.6e-7; with all six products in one sum twice as much.
    assert float((plain - ref).norm() / ref.norm()) < 2.0 ** -24 * (1 + ((H + 31) // 32) ** 0.5)
    largest, nan = rows // 2, rows + rows // 2
    x[largest, 5] = torch.finfo(torch.float32).max  # no finite bf16 is as large; times 2e-38 it is an ordinary number
    x[nan, 7] = float("nan")
    got, ref = run(), reference()
    keep = torch.ones(2 * rows, dtype=torch.bool, device="cuda")
    keep[[largest, nan]] = False
    assert torch.equal(got[keep], plain[keep])
    assert float((got[largest] - ref[largest]).norm() / ref[largest].norm()) < 1e-5  # sums in fp32, as above
    assert bool(got[nan].isnan().all())
    x[nan, 7] = float("inf")  # h is inf, -inf or (where the gate is -inf) NaN
    z, w = x[nan].double() @ g.double(), x[nan].double() @ u.double()
    h = torch.nn.functional.silu(z) * w
    y = h @ d.double()
    got = run()[nan]
    assert torch.equal(got.isnan(), y.isnan()) and torch.equal(got[~y.isnan()].double(), y[~y.isnan()])
    L.close()


# Numbers whose bf16 parts are denormal lose bits in them: outputs that those bits could show in are sums of fp32 products
# instead.  Powers of two on x and the weights, by column of x where `column`, that leave ordinary outputs or small ones.
@pytest.mark.parametrize("x_exp,gate_exp,up_exp,down_exp,column", [
    (127, -127, -127, 0, True), (118, -118, -118, 0, True), (118, -118, -118, 0, False), (-118, 118, 118, 0, False),
    (-109, 109, 109, 0, False), (0, 0, 0, -120, False), (0, 0, 0, -109, False), (-60, -60, 60, 121, False)])
@pytest.mark.parametrize("H,I,rows", [(40, 64, 1), (96, 100, 65), (1024, 512, 33)])
def test_fp32_small_numbers(H, I, rows, x_exp, gate_exp, up_exp, down_exp, column):
    gen = torch.Generator(device="cuda").manual_seed(11)
    cfg = SimpleNamespace(T=2 * rows, H=H, E=2, k=1, I=I, I_shared=0, n_ranks=2, slots_per_rank=1, max_replicas=1,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="fp32")
    L = ReviveLayer(cfg)
    g, u, d = (torch.randn(*s, generator=gen, device="cuda") * s[0] ** -0.5 for s in ((H, I), (H, I), (I, H)))
    x = torch.empty(2 * rows, H, device="cuda").uniform_(0.6, 0.9, generator=gen) * torch.randn(2 * rows, H, generator=gen, device="cuda").sign()
    at = slice(5, 6) if column else slice(None)
    for t, e in ((x[:, at], x_exp), (g[at], gate_exp), (u[at], up_exp), (d, down_exp)):
        t.ldexp_(torch.tensor(e, device="cuda"))
    zero, dead = rows // 2, 7  # a row of zeros among the others, an output that only zero weights go into
    x[zero] = 0
    g[:, dead] = u[:, dead] = 0
    packed = pack_expert(g, u, d)
    L.set_expert_weights([packed[0]] * 2, [packed[1]] * 2)
    y = L.empty(2 * rows, H).fill_(-7.0)
    L.expert_ffn(x, torch.tensor([0, rows, 2 * rows], dtype=torch.int32, device="cuda"), 2 * rows, out=(y, None))
    # h is held in fp32, like the kernel's: its denormal values are what the down projection is given
    h = (torch.nn.functional.silu(x.double() @ g.double()) * (x.double() @ u.double())).float().double()
    ref = h @ d.double()
    assert float(ref[1].norm()) > 0 and bool((y[zero] == 0).all())
    scale = 2.0 ** -min(down_exp, 0)  # small outputs
    y, ref = y.double() * scale, ref * scale
    # sums of up to 1024 fp32 products, each rounded by 2^-24 of a partial sum: 2^-24 sqrt(1024), in three products
    assert float((y - ref).norm() / ref.norm()) < 3 * 2.0 ** -24 * max(H, I) ** 0.5
    L.close()


# Rows that go through sums in fp32, a batch of nothing else and one row of many, do not make a call many times as long:
# 1.1 to 2.8 times were measured, 12 to 93 with one lane per output.
@pytest.mark.parametrize("value", [float("nan"), float("inf"), 2.0 ** -115])
@pytest.mark.parametrize("whole", [True, False])
def test_fp32_time_of_numbers_without_parts(value, whole):
    P, rows, H, I = 16, 64, 1024, 512
    N = P * rows
    gen = torch.Generator(device="cuda").manual_seed(12)
    cfg = SimpleNamespace(T=N, H=H, E=P, k=1, I=I, I_shared=0, n_ranks=P, slots_per_rank=1, max_replicas=1, score_fn="softmax",
                          n_group=1, topk_group=1, dtype="fp32")
    L = ReviveLayer(cfg)
    L.set_expert_weights(list(torch.randn(P, 2 * I, H, generator=gen, device="cuda")), list(torch.randn(P, H, I, generator=gen, device="cuda")))
    x, y = torch.randn(N, H, generator=gen, device="cuda"), L.empty(N, H)
    off = torch.arange(0, N + 1, rows, dtype=torch.int32, device="cuda")
    other = x.clone()
    other[slice(None) if whole else N // 2] *= value

    def us(rows):
        L.expert_ffn(rows, off, N, out=(y, None))
        times = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            L.expert_ffn(rows, off, N, out=(y, None))
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert us(other) < 5 * us(x)
    L.close()


# The kernels that share the work by rows per slot give the same bits: a whole batch and its microbatches may take
# different ones.  The same slots with other slots beside them: weights streamed, row-tiles of up to 256, of up to 320
# rows; the shared expert in the same calls and alone.
@pytest.mark.parametrize("H,I", [(64, 64), (256, 192), (704, 320), (1088, 448), (7168, 2048)])
def test_kernels_agree_bit_for_bit(H, I):
    gen = torch.Generator(device="cuda").manual_seed(7)

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(torch.bfloat16)

    def expert():
        return pack_expert(normal(H, I, std=H ** -0.5), normal(H, I, std=H ** -0.5), normal(I, H, std=I ** -0.5))

    own = [expert() if c else (None, None) for c in EDGES]
    other, sh = expert(), expert()
    n = sum(EDGES)
    x = normal(n, H)
    ref = None
    for streamed, beside in ((True, [0] * 90), (False, [200] * 8), (False, [320] * 120)):
        counts = EDGES + beside
        P, N = len(counts), sum(counts)
        assert (N <= 16 * P) == streamed and (streamed or N > 96 * P) and (beside[0] < 320 or N >= 128 * P)  # the rules' limits
        cfg = SimpleNamespace(T=N, H=H, E=P, k=1, I=I, I_shared=I, n_ranks=P, slots_per_rank=1, max_replicas=1,
                              score_fn="softmax", n_group=1, topk_group=1, dtype="bf16")
        L = ReviveLayer(cfg)
        packed = own + [other if c else (None, None) for c in beside]
        L.set_expert_weights([p[0] for p in packed], [p[1] for p in packed])
        xs = torch.cat([x, normal(N - n, H)])
        off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
        L.set_kernel_timing(True)
        y, y_sh = L.expert_ffn(xs, off, N, x=xs, w_sh_gate_up=sh[0], w_sh_down=sh[1])
        assert (L.kernel_times()["ffn_tiles"][1] == 0) == streamed
        got = [y[:n], y_sh[:n]]
        if ref is None:
            ref = got
        for a, b in zip(got, ref):
            assert torch.equal(a, b), (streamed, beside[0])
        for T in (1, 64, 65, 128, 129, 600, n):
            assert torch.equal(L.shared_ffn(xs[:T].contiguous(), sh[0], sh[1], T), ref[1][:T]), T
        L.close()


# Which kernel a layer takes (the one with 256-row tiles needs a list of them), at both sides of each limit: rows per
# slot, slots of little work, a shared expert that outweighs the slots (cached and not).
@pytest.mark.parametrize("P,H,I,I_shared,N,streamed", [
    (64, 256, 128, 0, 1024, True), (64, 256, 128, 0, 1025, False), (64, 1024, 576, 0, 6144, True), (64, 1024, 576, 0, 6145, False),
    (640, 256, 128, 0, 256, True), (641, 256, 128, 0, 256, False), (768, 256, 128, 0, 257, True), (769, 256, 128, 0, 800, False),
    (768, 448, 128, 0, 800, True), (800, 448, 128, 0, 800, False), (800, 704, 64, 0, 800, True),
    (800, 448, 192, 0, 800, True), (800, 448, 192, 0, 256, False), (800, 704, 128, 0, 64, True), (800, 704, 128, 0, 65, False),
    (300, 256, 128, 4096, 4096, True), (300, 256, 128, 2304, 4097, True), (300, 256, 128, 2368, 4097, False),
    (72, 2048, 256, 16448, 1024, True), (72, 2048, 256, 16448, 1025, False)])
def test_limits_of_the_streaming_kernel(P, H, I, I_shared, N, streamed):
    gen = torch.Generator(device="cuda").manual_seed(8)
    w, w_sh = ([(torch.randn(*s, generator=gen, device="cuda") * s[0] ** -0.5).to(torch.bfloat16) for s in ((H, n), (H, n), (n, H))]
               for n in (I, I_shared or 64))
    gu, dn = pack_expert(*w)
    gu_sh, dn_sh = pack_expert(*w_sh) if I_shared else (None, None)
    cfg = SimpleNamespace(T=N, H=H, E=min(P, 512), k=1, I=I, I_shared=I_shared, n_ranks=P, slots_per_rank=1, max_replicas=2,
                          score_fn="softmax", n_group=1, topk_group=1, dtype="bf16")
    L = ReviveLayer(cfg)
    L.set_expert_weights([gu] * P, [dn] * P)  # one expert everywhere
    off = torch.linspace(0, N, P + 1, device="cuda").round().to(torch.int32)
    x = torch.randn(N, H, generator=gen, device="cuda").to(torch.bfloat16)
    L.set_kernel_timing(True)
    y, y_sh = L.expert_ffn(x, off, N, x=x, w_sh_gate_up=gu_sh, w_sh_down=dn_sh)
    assert (L.kernel_times()["ffn_tiles"][1] == 0) == streamed
    assert rel_err(f64(y), _reference(x.float().cpu(), w).double().numpy()) < TOL["bf16"]
    if I_shared:
        assert torch.equal(y_sh, L.shared_ffn(x, gu_sh, dn_sh, N))
        assert rel_err(f64(y_sh[:64]), _reference(x[:64].float().cpu(), w_sh).double().numpy()) < TOL["bf16"]
    L.close()


# The longest rows that 64 of them take 32-bit offsets for, and longer ones: rows 61 to 63 of a tile, of x and of the
# weights, lie 4 GiB and more behind its first, where 32 bits would read other rows.
@pytest.mark.parametrize("H", [(1 << 24) - 8, (1 << 24) + (1 << 20)])
def test_fp32_rows_of_64_mib(H):
    """x holds four elements of a row, at its ends and in the middle: a sum over H has four products, one over I 64 of them,
    and 1e-5 is twenty times fp32's error."""
    I, counts = 64, [64, 0, 17]
    N, at = sum(counts), [0, 5, (1 << 23) + 3, H - 1]
    gen = torch.Generator(device="cuda").manual_seed(9)
    cfg = SimpleNamespace(T=N, H=H, E=3, k=1, I=I, I_shared=0, n_ranks=3, slots_per_rank=1, max_replicas=2, score_fn="softmax",
                          n_group=1, topk_group=1, dtype="fp32")
    L = ReviveLayer(cfg)
    weights = [(torch.randn(2 * I, H, generator=gen, device="cuda"), torch.randn(H, I, generator=gen, device="cuda")) if c else (None, None)
               for c in counts]
    L.set_expert_weights([w[0] for w in weights], [w[1] for w in weights])
    own, x = torch.randn(N, len(at), generator=gen, device="cuda"), torch.zeros(N, H, device="cuda")
    for j, col in enumerate(at):
        x[:, col] = own[:, j]
    y = L.empty(N, H).fill_(float("nan"))
    off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    L.expert_ffn(x, off, N, out=(y, None))
    torch.cuda.synchronize()
    for p, c in enumerate(counts):
        rows = slice(int(off[p]), int(off[p]) + c)
        if not c:
            continue
        h = own[rows].double() @ torch.stack([weights[p][0][:, col] for col in at]).double()
        h = torch.nn.functional.silu(h[:, :I]) * h[:, I:]
        worst, largest = [], []
        for a in range(0, H, 1 << 20):  # a library's product over all of H has left rows of its result at zero
            ref = h @ weights[p][1][a:a + (1 << 20)].double().T
            worst.append((y[rows, a:a + (1 << 20)] - ref).abs().max())
            largest.append(ref.abs().max())
        assert float(torch.stack(worst).max() / torch.stack(largest).max()) < 1e-5, p
    L.close()
