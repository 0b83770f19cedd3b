"""heart_pool_qk of more bytes than the memory-side cache holds (block means written through, runs
of blocks on one XCD): the bits of the same heads pooled one at a time, which is below that size, and the means in 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# B, H, N, D, block, tokens between heads (layout [B, N, H, D]); H * N * B * D * 4 bytes lie just above 256 MiB
SHAPES = [(1, 17, 31001, 128, 128, False), (2, 9, 29999, 128, 64, False), (1, 17, 31001, 128, 128, True),
          (3, 7, 50001, 64, 64, False), (1, 5, 210001, 64, 128, False), (1, 1, 524289, 128, 128, False),
          (1, 33, 32001, 64, 128, True)]


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
