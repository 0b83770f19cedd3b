"""Attention launches that deal out the kept blocks of all rows in equal shares: against the launch of one
workgroup per row and the oracle, where shares begin and end in every way they can."""
import numpy as np
import pytest
import torch

import oracle
from heart_testlib import np_gpu, u16

pytestmark = pytest.mark.gpu


# rows: one; as few as two shares; groups of 256 rows with a remainder; the most there are (D = 64, block 64: 2560) and one
# head more than that, which has a plan.  kinds: uneven with rows of no and one block; no blocks at all; all blocks
@pytest.mark.parametrize("kind", ["uneven", "empty", "full"])
@pytest.mark.parametrize("B,H,Nb,D,block,tail", [(1, 1, 1, 128, 128, 5), (1, 1, 150, 64, 64, 0), (1, 1, 197, 64, 64, 0), (2, 3, 6, 128, 128, 78),
                                                 (1, 1, 200, 128, 64, 63), (2, 7, 67, 64, 128, 1), (1, 3, 171, 64, 64, 7),
                                                 (2, 20, 64, 64, 64, 0), (1, 41, 64, 64, 64, 33)])
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
