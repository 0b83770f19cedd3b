"""heart_mask_topp: with long rows the work of the refreshed heads is dealt out over the chip by their
rank among all heads.  At the edges of that dealing every refreshed head gets what it gets when all heads are
refreshed, bit for bit, and every other head keeps its mask, lists and counts."""
import numpy as np
import pytest
import torch

import oracle
from heart_testlib import np_gpu

pytestmark = pytest.mark.gpu


_want = {}


# long rows: one head, heads around the 64 that one look at the flags covers, the most heads that are dealt and
# one more; one exact number of row groups; short rows
@pytest.mark.parametrize("B,H,Nb", [(1, 1, 257), (2, 32, 272), (1, 65, 260), (1, 13, 300), (4, 64, 257), (1, 257, 257),
                                    (3, 43, 7)])
@pytest.mark.parametrize("which", ["none", "first", "last", "some", "all"])
@pytest.mark.parametrize("slices", [False, True])
def test_refreshed_heads_only(B, H, Nb, which, slices):
    import paper_2605_14513_amd as heart

    D, BH = 64, B * H
    rng = np.random.default_rng(BH * 100 + Nb)
    qblk, kblk = (rng.standard_normal((B, H, Nb, D)).astype(np.float32) for _ in range(2))
    tau = rng.uniform(0.5, 0.95, H).astype(np.float32)
    flags = np.zeros(BH, np.uint8)
    if which == "first":
        flags[0] = 1
    elif which == "last":
        flags[-1] = 7  # (any value but 0)
    elif which == "some":
        flags[rng.permutation(BH)[:(BH + 1) // 2]] = 1
    elif which == "all":
        flags[:] = 1
    print(f"B={B} H={H} Nb={Nb} {which} slices={slices}", flush=True)
    gq, gk, gt = np_gpu(qblk), np_gpu(kblk), np_gpu(tau)
    ws = None
    if slices:
        ws = torch.empty(heart.heart_mask_topp_workspace_bytes(B, H, Nb, D), dtype=torch.uint8, device="cuda")
    full = heart.heart_mask_topp(gq, gk, gt, workspace=ws)
    if (B, H, Nb) not in _want:
        _want[B, H, Nb] = oracle.topp(oracle.scores(qblk, kblk), tau)[0]
    assert np.array_equal(full[0].cpu().numpy(), _want[B, H, Nb])
    mask = torch.full((B, H, Nb, Nb), 9, dtype=torch.uint8, device="cuda")
    idx = torch.full((B, H, Nb, Nb), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((B, H, Nb), -5, dtype=torch.int32, device="cuda")
    heart.heart_mask_topp(gq, gk, gt, refresh=np_gpu(flags.reshape(B, H)), mask=mask, kept_idx=idx, kept_count=cnt,
                          workspace=ws)
    torch.cuda.synchronize()
    on = torch.from_numpy(flags.reshape(B, H) != 0).cuda()
    for got, want, untouched in ((mask, full[0], 9), (idx, full[1], -1), (cnt, full[2], -5)):
        assert torch.equal(got[on], want[on])
        assert (got[~on] == untouched).all()


def test_as_many_workgroups_as_a_launch_holds():
    """2^23 - 1 heads of one block: the last grid of 512-thread workgroups whose threads fit 32 bits."""
    import paper_2605_14513_amd as heart

    H = (1 << 23) - 1
    x = torch.ones((1, H, 1, 16), device="cuda")
    tau = torch.full((H,), 0.9, device="cuda")
    mask = torch.zeros((1, H, 1, 1), dtype=torch.uint8, device="cuda")
    idx, cnt = torch.full((1, H, 1, 1), -1, dtype=torch.int32, device="cuda"), mask[..., 0].int()
    print(f"H={H}", flush=True)
    heart.heart_mask_topp(x, x, tau, mask=mask, kept_idx=idx, kept_count=cnt)
    torch.cuda.synchronize()
    assert (mask == 1).all() and (idx == 0).all() and (cnt == 1).all()


# scores handed in: rows whose sum lies around the two that 32-bit masses hold, next to each other in every order, with ties, empty
# rows, negative scores, NaN and scores above one (which count as 0, 0 and 1); one slot a lane, several, all; an odd last row
@pytest.mark.parametrize("Nb", [1, 15, 64, 65, 255, 300, 1000])
def test_scores_of_any_sum(Nb):
    import paper_2605_14513_amd as heart

    H = 3
    rng = np.random.default_rng(Nb)
    s = rng.exponential(size=(1, H, Nb, Nb)) ** 3
    s[rng.random(s.shape) < 0.2] = 1.0  # ties
    s = s / s.sum(-1, keepdims=True) * rng.choice([0.0, 0.3, 1.0, 1.89, 1.91, 2.1, 8.0, 300.0], size=(1, H, Nb, 1))
    s = s.astype(np.float32)
    counts = s.clip(0.0, 1.0)
    low = rng.random(s.shape) < 0.05
    given = np.where(low, np.where(rng.random(s.shape) < 0.5, np.float32(np.nan), np.float32(-0.5)), s)
    counts[low] = 0.0
    tau = np.array([0.4, 0.9, 0.999], np.float32)
    for keep in (1, 5):
        m, i, c = (x.cpu().numpy() for x in heart.heart_mask_topp(None, None, np_gpu(tau), scores_in=np_gpu(given), min_keep=keep))
        om, oi, oc = oracle.topp(counts, tau, min_keep=keep)
        assert np.array_equal(m, om) and np.array_equal(c, oc)
        listed = np.arange(Nb) < oc[..., None]
        assert np.array_equal(i[listed], oi[listed])


# the largest masses there are: every score counts as one, and the first half of the blocks has half of the mass.  One slot a lane and
# 32, beside a row without mass
@pytest.mark.parametrize("Nb", [31, 64, 257, 1024])
def test_scores_all_above_one(Nb):
    import paper_2605_14513_amd as heart

    s = torch.full((1, 1, Nb, Nb), 3.0, device="cuda")
    s[0, 0, 1::2] = 0.0
    print(f"scores all above one Nb={Nb}", flush=True)
    m, i, c = (x.cpu().numpy()[0, 0] for x in heart.heart_mask_topp(None, None, torch.full((1,), 0.5, device="cuda"), scores_in=s))
    half = (Nb + 1) // 2
    assert (c[::2] == half).all() and (c[1::2] == 1).all()
    assert (m[::2] == (np.arange(Nb) < half)).all() and (i[::2, :half] == np.arange(half)).all()
