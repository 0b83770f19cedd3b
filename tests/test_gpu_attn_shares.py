"""Attention launches that deal out the kept blocks of all rows in equal shares: against the launch of one
workgroup per row and the oracle, where shares begin and end in every way they can."""
import numpy as np
import pytest
import torch

import oracle
from heart_testlib import np_gpu, u16

pytestmark = pytest.mark.gpu


# rows: one; as few as two shares; groups of 256 rows with a remainder; the most there are in heads of 64 blocks at D = 64,
# block 64 (2560) and one head more than that, which has a plan; at D = 128 more rows than places (512, 1024 of the small
# workgroups), so that a share ends a row that another began, takes whole ones and begins the next, and two rows a place (more:
# below).  kinds: uneven with rows of no and one block; no blocks at all; all blocks
@pytest.mark.parametrize("kind", ["uneven", "empty", "full"])
@pytest.mark.parametrize("B,H,Nb,D,block,tail", [(1, 1, 1, 128, 128, 5), (1, 1, 150, 64, 64, 0), (1, 1, 197, 64, 64, 0), (2, 3, 6, 128, 128, 78),
                                                 (1, 1, 200, 128, 64, 63), (2, 7, 67, 64, 128, 1), (1, 3, 171, 64, 64, 7),
                                                 (2, 20, 64, 64, 64, 0), (1, 41, 64, 64, 64, 33),
                                                 (1, 6, 88, 128, 128, 40), (1, 7, 146, 128, 128, 0), (1, 21, 74, 128, 64, 9)])
def test_shares_of_rows(B, H, Nb, D, block, tail, kind):
    import paper_2605_14513_amd as heart

    N = Nb * block - tail
    rng = np.random.default_rng(Nb * 131 + D)
    cnt = rng.integers(0, Nb // 4 + 2, size=(B, H, Nb)).astype(np.int32).clip(0, Nb)
    cnt[rng.random(cnt.shape) < 0.1] = Nb
    cnt[0, 0, :3] = (Nb, 0, 1)[:Nb]
    if kind != "uneven":
        cnt[:] = Nb if kind == "full" else 0
    idx = np.broadcast_to(np.arange(Nb, dtype=np.int32), (B, H, Nb, Nb)).copy()
    if kind == "uneven":
        idx = rng.permuted(idx, axis=-1)
    g = torch.Generator(device="cuda").manual_seed(Nb)
    q, k, v = (torch.randn((B, N, H, D), generator=g, device="cuda").bfloat16().transpose(1, 2) for _ in range(3))
    gi, gc = np_gpu(idx), np_gpu(cnt)
    n_bytes = heart.heart_attn_balanced_workspace_bytes(q, block)
    shared = n_bytes > heart.heart_attn_workspace_bytes(q, block)
    assert shared == (B * H * Nb <= 2560 and Nb != 150)  # (2.5 rows a place; six parts of 25 blocks each are left as they are)
    print(f"B={B} H={H} Nb={Nb} D={D} block={block} {kind}", flush=True)
    for flags in (0, heart.HEART_ATTN_FOLD_SCALE):
        ws = torch.full((n_bytes + 64,), 255, dtype=torch.uint8, device="cuda")  # (NaN where nothing is written)
        lse, lse0 = (torch.full((B, H, N), float("nan"), device="cuda") for _ in range(2))
        out = torch.full_like(q, float("nan"))
        heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws[:n_bytes], flags=flags, lse=lse, out=out)
        one = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=None, flags=flags, lse=lse0)
        again = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws[:n_bytes], flags=flags)
        torch.cuda.synchronize()
        assert (ws[n_bytes:] == 255).all()
        assert torch.equal(out, again)
        if not shared:
            usual = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace="auto", flags=flags)
            assert torch.equal(out, usual)
            if Nb != 150:  # (a plan; those are split rows)
                assert torch.equal(out, one)
        empty = torch.isinf(lse0)
        assert torch.equal(torch.isinf(lse), empty)
        if not empty.all():
            assert (lse - lse0)[~empty].abs().max() <= 2e-5 * lse0[~empty].abs().max()
        # the same products and bf16 weights, whose sums start from other reference exponents: a weight moves by at
        # most two roundings (2^-8 of it in all), the output by one (2^-8); a tenth more for fp32
        mass = heart.heart_block_sparse_attn(q, k, v.abs(), block, gi, gc, workspace=None, flags=flags).float()
        bound = 1.1 * 2.0 ** -8 * (mass + one.float().abs()) * 1.01
        assert ((out.float() - one.float()).abs() <= bound).all()
        if N * H * B <= 20000 and kind == "uneven" and not flags:
            want = np.nan_to_num(oracle.attn(u16(q.contiguous()), u16(k.contiguous()), u16(v.contiguous()), block, idx, cnt))
            assert np.abs(out.float().cpu().numpy() - want).max() <= 2e-2 * max(1.0, np.abs(want).max() / 2)


# only the size that asks for it divides rows: a larger buffer, kept for several shapes, has the launch and the bits of
# heart_attn_workspace_bytes (the first shape has a plan, the second split rows)
@pytest.mark.parametrize("H,Nb,D,block", [(7, 67, 128, 128), (1, 200, 128, 64)])
def test_larger_workspaces_do_not_divide_rows(H, Nb, D, block):
    import paper_2605_14513_amd as heart

    rng = np.random.default_rng(Nb)
    cnt = rng.integers(1, Nb // 2, size=(1, H, Nb)).astype(np.int32)
    idx = np.broadcast_to(np.arange(Nb, dtype=np.int32), (1, H, Nb, Nb)).copy()
    g = torch.Generator(device="cuda").manual_seed(Nb)
    q, k, v = (torch.randn((1, H, Nb * block, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    gi, gc = np_gpu(idx), np_gpu(cnt)
    asked, usual = heart.heart_attn_balanced_workspace_bytes(q, block), heart.heart_attn_workspace_bytes(q, block)
    assert asked > usual
    print(f"H={H} Nb={Nb} D={D} block={block}", flush=True)
    ws = torch.empty(2 * asked, dtype=torch.uint8, device="cuda")
    want, divided = (heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws[:n]) for n in (usual, asked))
    assert not torch.equal(divided, want)  # (sums in another order)
    for n in (asked - 16, asked + 16, 2 * asked):
        assert torch.equal(heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws[:n]), want), n


# rows of 84 blocks, cut in five parts each ("parts": one head), in some twenty with short rows around them ("few"), and, with more
# rows than places, by shares ("shares": six heads)
@pytest.mark.parametrize("kind,H", [("parts", 1), ("few", 1), ("shares", 6)])
@pytest.mark.parametrize("flags", [0, 1])
def test_divided_rows_show_non_finite_inputs(kind, H, flags):
    """A NaN or an infinity that reaches a row of the undivided launch reaches it in the divided one, and no other row."""
    import paper_2605_14513_amd as heart

    Nb, D, block = 88, 128, 128
    N = Nb * block
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    blk = lambda i: slice(i * block, (i + 1) * block)
    nan_k, neg_k, inf_v, low = 30, 51, 70, 12  # key blocks that only some rows keep
    k[0, 0, blk(nan_k).start + 3] = float("nan")
    k[0, 0, blk(neg_k), 0] = float("-inf")
    v[0, 0, blk(inf_v), 2] = float("inf")
    k[0, 0, blk(low), 1], v[0, 0, blk(low), 2] = -400.0, float("nan")
    q[0, 0, blk(0).start + 5] = float("nan")
    q[0, 0, blk(2), 0] = q[0, 0, blk(3), 0] = 1.0
    q[0, 0, blk(4), 0] = -1.0
    q[0, 0, blk(6), 1] = 8.0
    plain = [j for j in range(Nb) if j not in (nan_k, neg_k, inf_v, low)]
    first = [plain, sorted(plain + [nan_k]), sorted(plain + [neg_k]), [neg_k], sorted(plain + [neg_k]), sorted(plain + [inf_v]),
             sorted(plain + [low]), plain]
    idx, cnt = np.zeros((1, H, Nb, Nb), np.int32), np.zeros((1, H, Nb), np.int32)
    for h in range(H):
        for i in range(Nb):
            r = first[i] if h == 0 and i < len(first) else plain if kind == "parts" else [plain[(h + i) % len(plain)]]
            idx[0, h, i, :len(r)], cnt[0, h, i] = r, len(r)
    gi, gc = np_gpu(idx), np_gpu(cnt)
    n_bytes = heart.heart_attn_balanced_workspace_bytes(q, block)
    assert n_bytes > heart.heart_attn_workspace_bytes(q, block)
    print(f"non-finite {kind} H={H} flags={flags}", flush=True)
    res = []
    for ws in (torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda"), None):
        lse = torch.empty((1, H, N), device="cuda")
        out = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws, flags=flags, lse=lse)
        res.append((out.float().cpu().numpy()[0], lse.cpu().numpy()[0]))
    (out, lse), (one, lse1) = res
    for h in range(H):
        for i in range(Nb):
            a, b = out[h, blk(i)], one[h, blk(i)]
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b)), f"row {h} {i}"
            assert np.array_equal(np.isneginf(lse[h, blk(i)]), np.isneginf(lse1[h, blk(i)])), f"row {h} {i}: lse"
    # what the rows above must show, whichever launch
    one = one[0]
    assert np.isnan(one[blk(0)][5]).all() and np.isfinite(np.delete(one[blk(0)], 5, 0)).all()
    assert np.isnan(one[blk(1)]).all() and np.isfinite(one[blk(2)]).all() and (one[blk(3)] == 0).all()
    assert np.isnan(one[blk(4)]).all() and not np.isfinite(one[blk(5)][:, 2]).any()
    assert np.isnan(one[blk(6)][:, 2]).all() and np.isfinite(one[7 * block:]).all()


# counts outside of [0, Nb] count as its ends: in the search for a share as in the row itself
@pytest.mark.parametrize("H,Nb,D,block", [(1, 200, 128, 64), (6, 88, 128, 128), (20, 64, 64, 64)])
def test_divided_rows_clamp_the_counts(H, Nb, D, block):
    import paper_2605_14513_amd as heart

    rng = np.random.default_rng(H)
    cnt = rng.integers(-3, Nb + 6, size=(1, H, Nb)).astype(np.int32)
    cnt[0, 0, :2], cnt[0, -1, -2:] = (-3, Nb + 5), (Nb + 5, -3)
    idx = rng.permuted(np.broadcast_to(np.arange(Nb, dtype=np.int32), (1, H, Nb, Nb)), axis=-1)
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, Nb * block, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    ws = torch.empty(heart.heart_attn_balanced_workspace_bytes(q, block), dtype=torch.uint8, device="cuda")
    assert ws.numel() > heart.heart_attn_workspace_bytes(q, block)
    print(f"clamped counts H={H} Nb={Nb} D={D} block={block}", flush=True)
    got, want = (heart.heart_block_sparse_attn(q, k, v, block, np_gpu(idx), np_gpu(c), workspace=ws)
                 for c in (cnt, cnt.clip(0, Nb)))
    assert torch.equal(got, want)


def test_divided_rows_in_a_captured_graph():
    """Captured once, replayed on other counts each time (other rows are divided elsewhere): the eager bits."""
    import paper_2605_14513_amd as heart

    H, Nb, D, block = 6, 88, 128, 128
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, H, Nb * block, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    idx = torch.arange(Nb, dtype=torch.int32, device="cuda").expand(1, H, Nb, Nb).contiguous()
    counts = [torch.randint(0, Nb // d, (1, H, Nb), generator=g, dtype=torch.int32, device="cuda") for d in (2, 8, 1, 2)]
    cnt, out = counts[0].clone(), torch.empty_like(q)
    n_bytes = heart.heart_attn_balanced_workspace_bytes(q, block)
    ws, ws2 = (torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda") for _ in range(2))

    def call():
        heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, out=out, workspace=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    for i, c in enumerate(counts):
        want = heart.heart_block_sparse_attn(q, k, v, block, idx, c, workspace=ws2)
        cnt.copy_(c)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        print(f"replay {i}", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {i}"


# parts that are added up where the last of them is left (two split parts; shares, of which the first shape has rows of three and
# more parts): whatever the workspace holds, eagerly and in replays, in between other calls with the same memory
@pytest.mark.parametrize("H,Nb,D,block", [(2, 5, 128, 128), (18, 11, 128, 128), (40, 10, 64, 64), (6, 88, 128, 64), (20, 64, 64, 64)])
def test_merged_parts_in_memory_of_any_contents(H, Nb, D, block):
    import paper_2605_14513_amd as heart

    N = Nb * block - 3
    rng = np.random.default_rng(H)
    cnt = np_gpu(rng.integers(Nb // 2, Nb + 1, size=(1, H, Nb)).astype(np.int32))
    idx = torch.arange(Nb, dtype=torch.int32, device="cuda").expand(1, H, Nb, Nb).contiguous()
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    ws = torch.zeros(heart.heart_attn_balanced_workspace_bytes(q, block), dtype=torch.uint8, device="cuda")
    out, lse = torch.empty_like(q), torch.empty((1, H, N), device="cuda")

    def call():
        heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, out=out, lse=lse, workspace=ws)

    print(f"merged H={H} Nb={Nb} D={D} block={block}", flush=True)
    call()
    want, want_lse = out.clone(), lse.clone()
    one = heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, workspace=None)
    mass = heart.heart_block_sparse_attn(q, k, v.abs(), block, idx, cnt, workspace=None).float()
    # (two roundings of a weight, one of the output, a tenth more for fp32: as above)
    assert ((want.float() - one.float()).abs() <= 1.1 * 2.0 ** -8 * (mass + one.float().abs()) * 1.01).all()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    for i in range(6):
        if i % 3 == 0:
            ws.fill_(0 if i else 255)
        elif i % 3 == 1:
            ws.copy_(torch.randint(0, 256, ws.shape, generator=g, dtype=torch.uint8, device="cuda"))
        for run in (call, graph.replay):
            out.fill_(float("nan"))
            lse.fill_(float("nan"))
            run()
            torch.cuda.synchronize()
            assert torch.equal(out, want) and torch.equal(lse, want_lse), f"round {i}"


def _bits_or_bound(heart, q, k, v, block, idx, cnt, ws, same):
    """A divided launch twice, whatever the workspace holds: the bits of the undivided one (`same`), or two roundings of a weight
    and one of the output from it (a tenth more for fp32, as above); the row sums that the two make."""
    B, H, N, _ = q.shape
    lse, lse0 = (torch.full((B, H, N), float("nan"), device="cuda") for _ in range(2))
    one = heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, workspace=None, lse=lse0)
    mass = heart.heart_block_sparse_attn(q, k, v.abs(), block, idx, cnt, workspace=None).float()
    for fill in (255, 0):
        ws.fill_(fill)
        out = heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, workspace=ws, lse=lse, out=torch.full_like(q, float("nan")))
        again = heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, again)
        if same:
            assert torch.equal(out, one) and torch.equal(lse, lse0)
        else:
            assert ((out.float() - one.float()).abs() <= 1.1 * 2.0 ** -8 * (mass + one.float().abs()) * 1.01).all()
            empty = torch.isinf(lse0)
            assert torch.equal(torch.isinf(lse), empty)
            assert empty.all() or (lse - lse0)[~empty].abs().max() <= 2e-5 * lse0[~empty].abs().max()
    return torch.equal(out, one)


def _lists(H, Nb, D, block, seed):
    N = Nb * block - 5
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn((1, N, H, D), generator=g, device="cuda").bfloat16().transpose(1, 2) for _ in range(3))
    idx = torch.argsort(torch.rand((1, H, Nb, Nb), generator=g, device="cuda"), dim=-1).int()
    return q, k, v, idx


# three to eight rows a place, where the heads are short (the most rows there are: 4096): shares that end a row, take several whole
# ones and begin the next
@pytest.mark.parametrize("kind", ["uneven", "long", "full", "empty"])
@pytest.mark.parametrize("H,Nb,D,block", [(26, 80, 128, 128), (16, 110, 128, 128), (8, 172, 128, 128), (256, 16, 128, 128),
                                          (585, 7, 128, 128), (14, 128, 128, 64), (8, 180, 64, 128), (3, 460, 64, 128),
                                          (512, 8, 64, 128), (50, 80, 64, 64), (16, 176, 64, 64)])
def test_shares_of_several_rows_a_place(H, Nb, D, block, kind):
    import paper_2605_14513_amd as heart

    q, k, v, idx = _lists(H, Nb, D, block, Nb)
    rng = np.random.default_rng(H)
    cnt = rng.integers(0, Nb // 4 + 2, size=(1, H, Nb)).clip(0, Nb).astype(np.int32)
    if kind == "long":
        cnt[rng.random(cnt.shape) < 0.1] = Nb
    elif kind != "uneven":
        cnt[:] = Nb if kind == "full" else 0
    n_bytes = heart.heart_attn_balanced_workspace_bytes(q, block)
    assert n_bytes > heart.heart_attn_workspace_bytes(q, block)
    print(f"H={H} Nb={Nb} D={D} block={block} {kind}", flush=True)
    ws = torch.empty(n_bytes, dtype=torch.uint8, device="cuda")
    _bits_or_bound(heart, q, k, v, block, idx, np_gpu(cnt), ws, same=False)


# most kept blocks of long heads that are divided: 7 / 25 of all, or as many a place (two workgroups a CU, four of the small ones), twice
# as many where an XCD has rows of one head at a time
def _most_divided(H, Nb, D, block):
    places, far = {(128, 128): (512, 225), (64, 64): (1024, 380), (128, 64): (1024, 96)}[D, block]
    return min(H * Nb * Nb * 7 // 25, (2 if H % 8 == 0 or 8 % H == 0 else 1) * far * places)


# lists of at most that many blocks are divided, others have the launch that a plan orders, and its bits
@pytest.mark.parametrize("H,Nb,D,block", [(3, 480, 128, 128), (4, 320, 128, 128), (3, 951, 64, 64), (2, 540, 128, 64),
                                          (8, 226, 128, 64), (1, 1100, 128, 64)])
def test_lists_that_keep_much_are_left_to_a_plan(H, Nb, D, block):
    import paper_2605_14513_amd as heart

    q, k, v, idx = _lists(H, Nb, D, block, Nb)
    rng = np.random.default_rng(H)
    most = _most_divided(H, Nb, D, block)
    ws = torch.empty(heart.heart_attn_balanced_workspace_bytes(q, block), dtype=torch.uint8, device="cuda")
    assert ws.numel() > heart.heart_attn_workspace_bytes(q, block)
    for total in (most // 2, most, most + 1, H * Nb * Nb):
        cnt = np.full(H * Nb, total // (H * Nb))
        move = rng.integers(0, cnt[0] + 1, H * Nb // 2)  # from one row to another
        cnt[:len(move)] -= move
        cnt[len(move):2 * len(move)] += move
        cnt[0] += total - cnt.sum()
        while (cnt > Nb).any():  # (what a row cannot hold goes to the shortest)
            i, j = cnt.argmax(), cnt.argmin()
            cnt[j], cnt[i] = cnt[j] + cnt[i] - Nb, Nb
        assert cnt.sum() == total and cnt.min() >= 0
        print(f"H={H} Nb={Nb} D={D} block={block} blocks={total} of {H * Nb * Nb}", flush=True)
        gc = np_gpu(cnt.astype(np.int32).reshape(1, H, Nb))
        same = _bits_or_bound(heart, q, k, v, block, idx, gc, ws, same=total > most)
        assert same == (total > most)


def test_divided_and_planned_lists_in_a_captured_graph():
    """Captured once, replayed on lists that are divided and on lists that are left to the plan: the eager bits."""
    import paper_2605_14513_amd as heart

    H, Nb, D, block = 4, 320, 128, 128
    q, k, v, idx = _lists(H, Nb, D, block, 1)
    g = torch.Generator(device="cuda").manual_seed(2)
    counts = [torch.randint(0, n, (1, H, Nb), generator=g, dtype=torch.int32, device="cuda") for n in (Nb // 2, Nb, Nb // 3, Nb, Nb // 2)]
    cnt, out = counts[1].clone(), torch.empty_like(q)
    n_bytes = heart.heart_attn_balanced_workspace_bytes(q, block)
    ws, ws2 = (torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda") for _ in range(2))

    def call():
        heart.heart_block_sparse_attn(q, k, v, block, idx, cnt, out=out, workspace=ws)

    call()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    for i, c in enumerate(counts):
        want = heart.heart_block_sparse_attn(q, k, v, block, idx, c, workspace=ws2)
        one = heart.heart_block_sparse_attn(q, k, v, block, idx, c, workspace=None)
        assert torch.equal(want, one) == (c.sum().item() > _most_divided(H, Nb, D, block))
        cnt.copy_(c)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        print(f"replay {i}", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {i}"


# rows split in two parts, which the workgroup that leaves the second adds up: what stands in either part, in both or in one without
# keys reaches the row, whichever of them comes last, and no other row
@pytest.mark.parametrize("H,Nb,D,block", [(18, 11, 128, 128), (40, 10, 64, 64), (34, 12, 128, 64), (20, 12, 64, 128)])
@pytest.mark.parametrize("flags", [0, 1])
def test_rows_in_two_parts_show_non_finite_inputs(H, Nb, D, block, flags):
    import paper_2605_14513_amd as heart

    N = Nb * block
    g = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    blk = lambda i: slice(i * block, (i + 1) * block)
    nan_k, neg_k, inf_v, nan_v = 0, 1, 2, 3  # key blocks that only some rows keep
    q[..., 0] = q[..., 0].abs() + 0.5        # (so the logits of block neg_k are -inf)
    k[0, :, blk(nan_k).start + 3] = float("nan")
    k[0, :, blk(neg_k), 0] = float("-inf")
    v[0, :, blk(inf_v), 2] = float("inf")
    v[0, :, blk(nan_v), 1] = float("nan")
    a, b, c, d = range(4, 8)  # blocks of finite values
    rows = [[a, b, c, d], [nan_k, a, b, c], [a, b, c, nan_k], [neg_k, neg_k, a, b], [a, b, neg_k, neg_k], [neg_k, neg_k], [neg_k],
            [inf_v, a, b, c], [a, b, inf_v, c], [nan_v, a]][:Nb - 2] + [[], [a]]
    idx, cnt = np.zeros((1, H, Nb, Nb), np.int32), np.zeros((1, H, Nb), np.int32)
    for h in range(H):
        for i in range(Nb):
            r = rows[(h + i) % len(rows)]
            idx[0, h, i, :len(r)], cnt[0, h, i] = r, len(r)
    gi, gc = np_gpu(idx), np_gpu(cnt)
    print(f"two parts H={H} Nb={Nb} D={D} block={block} flags={flags}", flush=True)
    n_bytes = heart.heart_attn_workspace_bytes(q, block)
    # (room for two parts a row)
    assert n_bytes == 2 * H * Nb * (block // 32) * (32 * D + 128) * 4
    res = []
    for fill in (255, 0, None):
        ws = None if fill is None else torch.full((n_bytes,), fill, dtype=torch.uint8, device="cuda")
        lse = torch.empty((1, H, N), device="cuda")
        out = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws, flags=flags, lse=lse)
        res.append((out.float().cpu().numpy()[0], lse.cpu().numpy()[0]))
    (out, lse), (out0, lse0), (one, lse1) = res
    assert np.array_equal(out, out0, equal_nan=True) and np.array_equal(lse, lse0, equal_nan=True)
    assert np.array_equal(np.isnan(out), np.isnan(one)) and np.array_equal(np.isinf(out), np.isinf(one))
    assert np.array_equal(np.isneginf(lse), np.isneginf(lse1)) and np.array_equal(np.isnan(lse), np.isnan(lse1))
    ok = np.isfinite(one)
    # (weights of at most four blocks of values below 6, two roundings of 2^-9 each and one of the output)
    assert np.abs(out[ok] - one[ok]).max() <= 1.1 * 2.0 ** -8 * 2 * 6
    for h in range(H):  # what the rows must show, whichever launch
        for i in range(Nb):
            r, x = rows[(h + i) % len(rows)], one[h, blk(i)]
            assert np.isnan(x).all() == (nan_k in r)
            assert (x == 0).all() == (set(r) <= {neg_k})
            assert np.isposinf(x[:, 2]).all() == (inf_v in r)
            assert np.isnan(x[:, 1]).all() == (nan_v in r or nan_k in r)
