"""heart_pool_qk of more bytes than the memory-side cache holds (block means written through, runs
of blocks on one XCD): the bits of the same heads pooled one at a time, which is below that size, and the means in 64 bits."""
import pytest
import torch

from heart_testlib import captured_functions

pytestmark = pytest.mark.gpu

# B, H, N, D, block, tokens between heads (layout [B, N, H, D]); H * N * B * D * 4 bytes lie just above 256 MiB, 384 with blocks of 32 KB
# (and, plain pass on both sides, above 256: see test_route)
SHAPES = [(1, 17, 31001, 128, 128, False), (2, 9, 29999, 128, 64, False), (1, 17, 31001, 128, 128, True),
          (3, 7, 50001, 64, 64, False), (1, 5, 210001, 64, 128, False), (1, 1, 524289, 128, 128, False),
          (1, 33, 32001, 64, 128, True), (1, 26, 31001, 128, 128, False), (1, 17, 31001, 128, 64, True),
          (1, 33, 31001, 128, 128, True), (101, 40, 130, 128, 64, False)]


@pytest.mark.parametrize("B,H,N,D,block,strided", SHAPES)
def test_large_call_has_the_bits_of_its_heads(B, H, N, D, block, strided):
    import paper_2605_14513_amd as heart

    print(f"pool B={B} H={H} N={N} D={D} block={block} strided={strided}", flush=True)
    assert 4 * B * H * N * D > 256 << 20
    gen = torch.Generator(device="cuda").manual_seed(N)
    shape = (B, N, H, D) if strided else (B, H, N, D)
    q, k = (torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    if strided:
        q, k = q.transpose(1, 2), k.transpose(1, 2)
    Nb = -(-N // block)
    got = heart.heart_pool_qk(q, k, block)
    for b in range(B):
        for h in range(H):
            one = heart.heart_pool_qk(q[b:b + 1, h:h + 1], k[b:b + 1, h:h + 1], block)
            for name, g, w in zip(("qblk", "kblk", "qmean", "kmean"), got, one):
                assert torch.equal(g[b, h], w[0, 0]), (name, b, h)
    # sums of at most 128 fp32 terms: |error| <= 128 * 2^-24 * sum|x| / n
    for x, blocks in ((q, got[0]), (k, got[1])):
        for h in (0, H - 1):
            pad = torch.zeros(Nb * block, D, dtype=torch.float64, device="cuda")
            pad[:N] = x[B - 1, h].double()
            n = torch.full((Nb, 1), float(block), dtype=torch.float64, device="cuda")
            n[-1] = N - (Nb - 1) * block
            rows = pad.view(Nb, block, D)
            err = (blocks[B - 1, h].double() - rows.sum(1) / n).abs()
            assert bool((err <= 2.0 ** -17 * rows.abs().sum(1) / n).all()), h


def tensors(B, H, N, D, strided):
    shape = (B, N, H, D) if strided else (B, H, N, D)
    return (torch.empty(shape, dtype=torch.bfloat16, device="cuda").transpose(1, 2) if strided
            else torch.empty(shape, dtype=torch.bfloat16, device="cuda"))


# either side of each limit: bytes, with blocks of 16 and of 32 KB; rows between those of other heads, which short heads and rows of
# D = 64 have read by the plain pass whatever the size (105 items of 40 heads of 130 tokens took 93 us in the place of 88)
@pytest.mark.parametrize("B,H,N,D,block,strided,stream", [
    (1, 17, 31001, 128, 64, False, True), (1, 16, 32768, 128, 64, False, False), (1, 17, 31001, 64, 128, False, False),
    (1, 33, 32001, 64, 128, False, True), (1, 24, 32768, 128, 128, False, False), (1, 26, 31001, 128, 128, False, True),
    (5, 40, 3000, 128, 128, False, False), (1, 17, 32760, 128, 128, True, False), (1, 31, 32001, 128, 128, True, True),
    (1, 17, 31001, 128, 64, True, True), (105, 40, 130, 128, 128, True, False), (46, 40, 500, 128, 64, True, False),
    (32, 40, 1999, 128, 128, True, False), (25, 40, 2000, 128, 128, True, True), (1, 70, 32001, 64, 64, True, False)])
def test_route(B, H, N, D, block, strided, stream):
    import paper_2605_14513_amd as heart

    print(f"pool route B={B} H={H} N={N} D={D} block={block} strided={strided}", flush=True)
    few = tensors(1, 2, 1000, D, False)
    plain = captured_functions(lambda: heart.heart_pool_qk(few, few, block))[0]
    x = tensors(B, H, N, D, strided)
    assert (captured_functions(lambda: heart.heart_pool_qk(x, x, block))[0] != plain) == stream


# one head: there is no call of fewer heads, but its parts of whole blocks are calls below the limit
def test_one_head_has_the_block_means_of_its_parts():
    import paper_2605_14513_amd as heart

    N, D, block = 800001, 128, 128
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k = (torch.randn((1, 1, N, D), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    print(f"pool one head N={N}", flush=True)
    got = heart.heart_pool_qk(q, k, block)
    for first in range(0, N, 3000 * block):
        part = slice(first, min(N, first + 3000 * block))
        for g, w in zip(got[:2], heart.heart_pool_qk(q[:, :, part], k[:, :, part], block)[:2]):
            assert torch.equal(g[:, :, first // block:first // block + w.shape[2]], w), first


# heart_pool_drift of such a call: the block and token means of heart_pool_qk, and what heart_drift makes of them
@pytest.mark.parametrize("B,H,N,D,block,strided", [(2, 9, 29999, 128, 64, False), (1, 26, 31001, 128, 128, False),
                                                   (1, 33, 31001, 128, 128, True), (3, 7, 50001, 64, 64, False)])
def test_drift_of_a_large_call(B, H, N, D, block, strided):
    import paper_2605_14513_amd as heart

    q, k = tensors(B, H, N, D, strided).normal_(), tensors(B, H, N, D, strided).normal_()
    f32 = dict(dtype=torch.float32, device="cuda")
    Nb = -(-N // block)
    outs = dict(qblk=torch.empty((B, H, Nb, D), **f32), kblk=torch.empty((B, H, Nb, D), **f32),
                qmean=torch.empty((B, H, D), **f32), kmean=torch.empty((B, H, D), **f32),
                drift=torch.empty((B, H), **f32), refresh=torch.empty((B, H), dtype=torch.uint8, device="cuda"))
    state = [torch.zeros((B, H, D), **f32), torch.zeros((B, H, D), **f32), torch.ones((B, H), dtype=torch.uint8, device="cuda")]
    other = [x.clone() for x in state]
    delta = torch.full((H,), 0.05, **f32)
    ws = torch.zeros(heart.heart_pool_drift_workspace_bytes(B, H), dtype=torch.uint8, device="cuda")
    print(f"pool drift B={B} H={H} N={N} D={D} block={block} strided={strided}", flush=True)
    heart.heart_pool_drift(q, k, block, *state, delta, ws, 0.2, 0.8, True, **outs)
    want = heart.heart_pool_qk(q, k, block)
    for name, w in zip(("qblk", "kblk", "qmean", "kmean"), want):
        assert torch.equal(outs[name], w), name
    drift, refresh = heart.heart_drift(want[2], want[3], *other, delta, 0.2, 0.8)
    assert torch.equal(outs["drift"], drift) and torch.equal(outs["refresh"], refresh)
    assert all(torch.equal(a, b) for a, b in zip(state, other))
