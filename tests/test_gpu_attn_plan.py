"""The launch plan of heart_block_sparse_attn at the edges of its per-head row orders: the batches of
similar kept lists against a plain model of the rule, and the same output bits in every order.  Launches
of few rows, whose lists are split over several workgroups, against the oracle and the unsplit launch."""
import numpy as np
import pytest
import torch

import oracle
from heart_testlib import check_attn_plan, np_gpu, u16

pytestmark = pytest.mark.gpu


def near_rows(idx, cnt, batch):
    """Rows of one head in launch order: the longest left (lower index first) and the batch - 1 rows
    nearest to it, in order of length; nearness = the list at eight evenly spaced ranks and four
    times the length, sum of absolute differences."""
    Nb = len(cnt)
    sig = np.zeros((Nb, 9), np.int64)
    for r in range(Nb):
        if cnt[r] > 0:
            sig[r, :8] = [idx[r, cnt[r] * (2 * k + 1) // 16] for k in range(8)]
        sig[r, 8] = 4 * cnt[r]
    left, out = np.argsort(-cnt.astype(np.int64), kind="stable"), []
    while len(left):
        d = np.abs(sig[left] - sig[left[0]]).sum(1)
        take = np.zeros(len(left), bool)
        take[np.argsort(d, kind="stable")[:batch]] = True
        out += left[take].tolist()
        left = left[~take]
    return np.array(out)


# rows per head at the ends of the range that has batches, around the register layouts (64 rows a
# slot: 256 / 257, 640 / 641) and ragged; heads around the two per XCD that are walked in turn
@pytest.mark.parametrize("H,Nb,block", [(17, 64, 64), (9, 63, 128), (16, 65, 64), (3, 256, 128), (5, 257, 64),
                                        (2, 640, 64), (2, 641, 64), (2, 1024, 64), (1, 1023, 128)])
def test_batches_of_similar_rows(H, Nb, block):
    import paper_2605_14513_amd as heart

    D = 64
    N = Nb * block - 3
    rng = np.random.default_rng(H * 10007 + Nb)
    cnt = rng.integers(0, min(Nb, 12) + 1, size=(1, H, Nb)).astype(np.int32)
    cnt[0, 0, :7] = Nb  # a few full rows, equal to each other
    idx = np.zeros((1, H, Nb, Nb), np.int32)
    for h in range(H):
        for i in range(Nb):
            idx[0, h, i, :cnt[0, h, i]] = np.sort(rng.permutation(Nb)[:cnt[0, h, i]])
    g = torch.Generator(device="cuda").manual_seed(Nb)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    gi, gc = np_gpu(idx), np_gpu(cnt)
    base = heart.heart_workspace_bytes(1, H, Nb, D) // 4
    full = heart.heart_attn_workspace_bytes(q, block) // 4
    near_words = H * Nb if 64 <= Nb <= 1024 else 0
    assert full == base + near_words + (2304 // 4 if H * Nb > 512 else 0)  # + counters a cache line apart
    print(f"H={H} Nb={Nb} block={block}", flush=True)
    outs = []
    for words in (full, base + near_words, base, None):
        ws = None if words is None else torch.full((words + 5,), -7, dtype=torch.int32, device="cuda")[:words]
        outs.append(heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws))
        torch.cuda.synchronize()
        if ws is None:
            continue
        check_attn_plan(ws.cpu().numpy(), cnt, Nb)
        n_wg = torch.cuda.get_device_properties(0).multi_processor_count * 2 * 128 // block
        if words >= base + near_words > base and H * Nb > n_wg:
            near = ws[base:base + near_words].cpu().numpy().reshape(H, Nb)
            batch = (n_wg + 7) // 8 * (2 if H <= 16 else 1)
            for h in range(H):
                assert np.array_equal(near[h], h * Nb + near_rows(idx[0, h], cnt[0, h], batch)), f"head {h}"
    assert all(torch.equal(outs[0], o) for o in outs[1:])


# parts per row with two workgroups per CU (block 128) or four; one head's places not divisible by the
# rows; both block sizes; token-major tensors; short last blocks; with `ramp` the logits of a block lie that many
# log2 units above (or below) those of the block before it, so that the parts' reference exponents lie
# 160 to 200 apart and all parts but the last, or the first, have no weight
@pytest.mark.parametrize("H,Nb,D,block,tail,parts,ramp", [
    (1, 8, 128, 128, 0, 2, 0), (1, 64, 128, 128, 5, 8, 0), (1, 67, 128, 64, 63, 15, 0), (3, 50, 128, 128, 127, 3, 0),
    (1, 64, 64, 64, 1, 16, 0), (3, 50, 64, 64, 0, 6, 0), (4, 9, 64, 128, 100, 2, 0), (1, 64, 128, 128, 5, 8, 25),
    (1, 64, 64, 64, 1, 16, 40), (1, 66, 128, 64, 17, 15, 40)])
def test_split_rows(H, Nb, D, block, tail, parts, ramp):
    import paper_2605_14513_amd as heart

    N = Nb * block - tail
    rng = np.random.default_rng(Nb * 131 + D)
    cnt = rng.integers(0, Nb + 1, size=(1, H, Nb)).astype(np.int32)
    cnt[0, 0, :4] = (0, 1, parts - 1, Nb)  # no, one, almost one key block a part, all
    if ramp:
        cnt[0, 0, 4:12] = Nb
    idx = np.zeros((1, H, Nb, Nb), np.int32)
    for h in range(H):
        for i in range(Nb):
            idx[0, h, i, :cnt[0, h, i]] = np.sort(rng.permutation(Nb)[:cnt[0, h, i]])
    idx[0, 0, 1, 0] = Nb - 1  # the short last block alone
    g = torch.Generator(device="cuda").manual_seed(Nb)
    q, k, v = (torch.randn((1, N, H, D), generator=g, device="cuda") for _ in range(3))
    if ramp:
        # rising, falling, and nearly level (parts that all have some weight)
        blk = torch.arange(N, device="cuda") // block
        q[..., 0] = torch.tensor([8.0, -8.0, 0.05], device="cuda")[blk % 3][None, :, None]
        k[..., 0] = (blk * (ramp * D ** 0.5 / (8 * 1.442695)))[None, :, None]
    q, k, v = (x.bfloat16().transpose(1, 2) for x in (q, k, v))
    gi, gc = np_gpu(idx), np_gpu(cnt)
    n_bytes = heart.heart_attn_workspace_bytes(q, block)
    # per part and 32 query rows: 32 x D accumulators and 64 lanes' softmax states, 4 bytes each
    assert n_bytes == 4 * parts * H * Nb * (block // 32) * (32 * D + 128)
    print(f"H={H} Nb={Nb} D={D} block={block} parts={parts} ramp={ramp}", flush=True)
    # (the oracle has no value for a row without blocks, the kernel zeros)
    want, mass = (np.nan_to_num(oracle.attn(u16(q.contiguous()), u16(k.contiguous()), u16(x.contiguous()), block, idx, cnt))
                  for x in (v, v.abs()))
    # The kernel rounds every weight to bf16 (by at most 2^-8 of it, so at most 2^-8 sum p|v| of an output) and the
    # output (2^-8 of it); a tenth more for fp32.  With a ramp the logits reach 1.4e4 before the scaling, where fp32
    # has steps of 2^-10: four of them in a sum move a weight by up to 4 * 2^-10 / sqrt(64).
    each = 1.1 * 2.0 ** -8 * (mass + np.abs(want)) + (5e-4 * mass if ramp else 0.0)
    for flags in (0, heart.HEART_ATTN_FOLD_SCALE):
        ws = torch.full((n_bytes + 64,), 255, dtype=torch.uint8, device="cuda")  # (NaN where nothing is written)
        lse, lse0 = (torch.full((1, H, N), float("nan"), device="cuda") for _ in range(2))
        out = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws[:n_bytes], flags=flags, lse=lse)
        one = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=None, flags=flags, lse=lse0)
        small = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws[:n_bytes - 16], flags=flags)
        torch.cuda.synchronize()
        assert (ws[n_bytes:] == 255).all()
        assert torch.equal(small, one)  # no room for the parts: the unsplit launch
        empty = torch.isinf(lse0)
        assert torch.equal(torch.isinf(lse), empty) and (lse - lse0)[~empty].abs().max() <= 2e-5 * lse0[~empty].abs().max()
        a, b = out.float().cpu().numpy(), one.float().cpu().numpy()
        assert (np.abs(a - b) <= 2.0 * each).all(), (np.abs(a - b) / np.maximum(each, 1e-30)).max()
        if flags and ramp:
            continue  # (the folded scale rounds the query's 8 and with it logits of 2^11: only the launches are compared)
        # each output; the folded scale rounds q as well, 2^-8 of every product of a logit (their absolute values
        # add up to about 0.64 sqrt(D), at most 8)
        bound = each + (8 * 2.0 ** -8 * mass if flags else 0.0)
        assert (np.abs(a - want) <= bound).all(), (np.abs(a - want) / np.maximum(bound, 1e-30)).max()
        # each row: the roundings are independent and a bf16 rounding is 1.6e-3 in the root mean square (2^-8 / sqrt(3),
        # over the values between two powers of two), so its relative error is about sqrt(2) of that, with the folded
        # scale sqrt(3); three times as much
        err, size = np.linalg.norm(a - want, axis=-1), np.linalg.norm(want, axis=-1)
        assert (err <= 3 * 1.63e-3 * (3 if flags else 2) ** 0.5 * size).all(), (err / np.maximum(size, 1e-30)).max()


# D = 128: eight parts of eight blocks; the small workgroups of blocks of 64: sixteen parts of four
@pytest.mark.parametrize("D,block", [(128, 128), (64, 64)])
@pytest.mark.parametrize("flags", [0, 1])
def test_split_rows_show_non_finite_inputs(D, block, flags):
    """A NaN or an infinity that reaches a row of the unsplit launch reaches it in the split one, also
    where it lies in one part alone or in one that has no weight; and no other row."""
    import paper_2605_14513_amd as heart

    Nb = 64
    N = Nb * block
    g = torch.Generator(device="cuda").manual_seed(D)
    q, k, v = (torch.randn((1, 1, N, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    blk = lambda i: slice(i * block, (i + 1) * block)
    nan_k, neg_k, inf_v, low = 20, 37, 51, 9  # key blocks that only some rows keep
    k[0, 0, blk(nan_k).start + 3] = float("nan")
    k[0, 0, blk(neg_k), 0] = float("-inf")
    v[0, 0, blk(inf_v), 2] = float("inf")
    k[0, 0, blk(low), 1], v[0, 0, blk(low), 2] = -400.0, float("nan")
    rows = [[j for j in range(Nb) if j not in (nan_k, neg_k, inf_v, low)] for _ in range(Nb)]
    q[0, 0, blk(0).start + 5] = float("nan")         # row 0: one query without a finite logit
    rows[1] = sorted(rows[1] + [nan_k])              # row 1: one key of NaN
    rows[2] = sorted(rows[2] + [neg_k])              # row 2: logits of -inf in one block
    rows[3] = [neg_k]                                # row 3: no other logits
    rows[4] = sorted(rows[4] + [neg_k])              # row 4: logits of +inf
    rows[5] = sorted(rows[5] + [inf_v])              # row 5: an infinite value
    rows[6] = sorted(rows[6] + [low])                # row 6: a value of NaN without weight
    q[0, 0, blk(2), 0] = q[0, 0, blk(3), 0] = 1.0
    q[0, 0, blk(4), 0] = -1.0
    q[0, 0, blk(6), 1] = 8.0                         # (logits 400 to 600 in log2 units lower)
    cnt = np.array([len(r) for r in rows], np.int32).reshape(1, 1, Nb)
    idx = np.zeros((1, 1, Nb, Nb), np.int32)
    for i, r in enumerate(rows):
        idx[0, 0, i, :len(r)] = r
    gi, gc = np_gpu(idx), np_gpu(cnt)
    res = []
    for n_bytes in (heart.heart_attn_workspace_bytes(q, block), heart.heart_workspace_bytes(1, 1, Nb, D)):
        ws = torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda")
        lse = torch.empty((1, 1, N), device="cuda")
        out = heart.heart_block_sparse_attn(q, k, v, block, gi, gc, workspace=ws, flags=flags, lse=lse)
        res.append((out.float().cpu().numpy()[0, 0], lse.cpu().numpy()[0, 0]))
    torch.cuda.synchronize()
    (out, lse), (one, lse1) = res
    for i in range(Nb):
        a, b = out[blk(i)], one[blk(i)]
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b)), f"row {i}"
        assert np.array_equal(np.isneginf(lse[blk(i)]), np.isneginf(lse1[blk(i)])), f"row {i}: lse"
    # what the rows above must show, whichever launch
    assert np.isnan(one[blk(0)][5]).all() and np.isfinite(np.delete(one[blk(0)], 5, 0)).all()
    assert np.isnan(one[blk(1)]).all() and np.isfinite(one[blk(2)]).all() and (one[blk(3)] == 0).all()
    assert np.isnan(one[blk(4)]).all() and not np.isfinite(one[blk(5)][:, 2]).any()
    assert np.isnan(one[blk(6)][:, 2]).all() and np.isfinite(one[7 * block:]).all()


def test_more_heads_than_plan_workgroups():
    """More heads than a launch of one 1024-thread workgroup per head can have (2^32 threads); every
    head has one row of one key, so its output is that key's value."""
    import paper_2605_14513_amd as heart

    H = (1 << 22) + 5
    v = torch.randn((1, H, 1, 64), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda",
                    dtype=torch.bfloat16)
    cnt = torch.ones((1, H, 1), dtype=torch.int32, device="cuda")
    cnt[0, 7::1001] = 0
    idx = torch.zeros((1, H, 1, 1), dtype=torch.int32, device="cuda")
    ws = torch.full((heart.heart_workspace_bytes(1, H, 1, 64) // 4,), -7, dtype=torch.int32, device="cuda")
    print(f"H={H}", flush=True)
    out = heart.heart_block_sparse_attn(v, v, v, 64, idx, cnt, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(out, v * cnt[..., None])
    # totals per head, then the only row of every head
    assert torch.equal(ws[24 + H:24 + 2 * H], cnt.view(-1))
    assert torch.equal(ws[24 + 2 * H:], torch.arange(H, dtype=torch.int32, device="cuda"))


# beyond 1024 heads: the heads are dealt out in turn and the row orders write the totals; rows too few for
# batches (small workgroups) and enough for them
@pytest.mark.parametrize("H,Nb", [(1025, 1), (1029, 9), (1100, 70)])
def test_plan_of_heads_that_are_not_ranked(H, Nb):
    import paper_2605_14513_amd as heart

    rng = np.random.default_rng(H)
    cnt = rng.integers(0, Nb + 1, size=(1, H, Nb)).astype(np.int32)
    idx = np.broadcast_to(np.arange(Nb, dtype=np.int32), (1, H, Nb, Nb))
    g = torch.Generator(device="cuda").manual_seed(H)
    v = torch.randn((1, H, Nb * 64 - 1, 64), generator=g, device="cuda", dtype=torch.bfloat16)
    gi, gc = np_gpu(idx), np_gpu(cnt)
    print(f"H={H} Nb={Nb}", flush=True)
    ref = heart.heart_block_sparse_attn(v, v, v, 64, gi, gc, workspace=None)
    classes = 31 - ((cnt[0].astype(np.int64) * ((31 << 16) // Nb)) >> 16)
    for words in (heart.heart_workspace_bytes(1, H, Nb, 64) // 4, heart.heart_attn_workspace_bytes(v, 64) // 4):
        ws = torch.full((words,), -7, dtype=torch.int32, device="cuda")
        out = heart.heart_block_sparse_attn(v, v, v, 64, gi, gc, workspace=ws)
        torch.cuda.synchronize()
        plan = ws.cpu().numpy()
        assert torch.equal(out, ref)
        assert np.array_equal(plan[24:24 + H], np.concatenate([np.arange(x, H, 8) for x in range(8)]))
        assert np.array_equal(plan[24 + H:24 + 2 * H], cnt[0].sum(1))
        seq = plan[24 + 2 * H:24 + 2 * H + H * Nb].reshape(H, Nb)
        want = np.arange(H)[:, None] * Nb + np.argsort(classes, axis=1, kind="stable")
        assert np.array_equal(seq, want)


# D = 128, blocks of 64: few rows of few heads use two workgroups a CU while less than 5/8 of the blocks are kept: on
# either side of that share, at the ends of the range of rows (the last size is beyond it) and of heads
@pytest.mark.parametrize("H,Nb,tail", [(1, 515, 63), (4, 150, 33), (2, 301, 0), (4, 768, 0), (5, 150, 1), (4, 769, 9)])
@pytest.mark.parametrize("share", ["few", "just below", "just above", "all"])
def test_workgroups_of_few_heads(H, Nb, tail, share):
    import paper_2605_14513_amd as heart

    D, block = 128, 64
    N = Nb * block - tail
    rng = np.random.default_rng(Nb)
    if share == "few":
        cnt = rng.integers(0, 10, size=(1, H, Nb)).astype(np.int32)
    else:
        cnt = np.full((1, H, Nb), Nb if share == "all" else Nb * 5 // 8, np.int32)
        if share != "all":
            more = (5 * H * Nb * Nb + 7) // 8 - cnt.sum() - (share == "just below")  # (8 kept >= 5 H Nb^2, or one less)
            cnt.reshape(-1)[:max(more, 0)] += 1
            cnt[0, 0, 0] += min(more, 0)
            assert (8 * int(cnt.sum()) >= 5 * H * Nb * Nb) == (share == "just above")
    idx = torch.arange(Nb, dtype=torch.int32, device="cuda").expand(1, H, Nb, Nb).contiguous()
    gc = np_gpu(cnt)
    g = torch.Generator(device="cuda").manual_seed(Nb)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda").bfloat16() for _ in range(3))
    print(f"H={H} Nb={Nb} {share}", flush=True)
    want = heart.heart_block_sparse_attn(q, k, v, block, idx, gc, workspace=None)
    for n_bytes in (heart.heart_attn_workspace_bytes(q, block), heart.heart_workspace_bytes(1, H, Nb, D)):
        ws = torch.full((n_bytes // 4,), -7, dtype=torch.int32, device="cuda")
        out = heart.heart_block_sparse_attn(q, k, v, block, idx, gc, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        check_attn_plan(ws.cpu().numpy(), cnt, Nb)
