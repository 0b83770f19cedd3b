"""Timed workloads of the sparse-attention path, through its public entry points.

A case is a dict of plain values.  `path` says which calls one pass makes:

  step    one sparse attention call of a layer in mid-generation (TmrDriver, drift policy): pool +
          drift -> top-p mask of the refreshed heads -> block-sparse attention
  dense   the same driver in its dense warm-up steps: attention over every key block
  attn    heart_block_sparse_attn(_flags) on lists that are there already: a step that reuses every mask
  refresh the mask-refresh side of a step alone: heart_pool_drift -> heart_mask_topp
  scores  the antidiagonal-style estimator and the selection from its scores, all heads
  ebc     the band error of one (head, candidate) of a threshold calibration

Inputs follow the recipe of `heart_synth` (per head four sinusoids over the latent grid times
directions that Q and K share, plus noise), generated on the GPU.  A `step` or `refresh` state
holds two denoising steps between which a bit over half of the heads move (the rest hardly) and
alternates between them, so that every pass refreshes the heads that moved and reuses the others,
as the passes of a generation do.
"""
from __future__ import annotations

import math

import torch

import paper_2605_14513_amd as heart
from paper_2605_14513_amd.tmr import SLICED_SCORES_MIN_NB, TmrConfig, TmrDriver

DELTA = 1.0          # drift threshold of the synthetic schedule
JUMP_SHARE = 0.55    # share of heads that move from one step to the next
GATE = (0.4, 0.8)    # layer gate of the method


def _case(name, path, B, H, T, Y, X, D, block, *, text=0, layout="bhnd", tau_lo=0.85, tau_hi=0.98,
          kept=0.25, fold=False, C=0):
    c = {"path": path, "B": B, "H": H, "T": T, "Y": Y, "X": X, "D": D, "block": block, "text": text,
         "layout": layout, "tau_lo": tau_lo, "tau_hi": tau_hi, "kept": kept, "fold": fold, "C": C}
    if name:
        c["name"] = name
    return c


def listed():
    # `kept`: share of the key blocks that the thresholds keep on these fields; only `work` reads it
    return [
        # the tiny configuration: launches and host time
        _case("step_tiny", "step", 1, 2, 4, 16, 16, 64, 64, kept=0.68),
        # two guidance branches, three heads, a short last block, token-major tensors as a
        # projection layer leaves them
        _case("step_small_ragged", "step", 2, 3, 3, 10, 23, 128, 128, layout="bnhd", kept=0.8),
        # head dimension 64 with blocks of 64: a mid-size clip, odd sizes
        _case("step_d64_b64", "step", 2, 10, 9, 23, 31, 64, 64, layout="bnhd", kept=0.30),
        # Wan2.1-1.3B and Wan2.1-14B at 480P: the ordinary sparse step
        _case("step_wan1p3b_480p", "step", 1, 12, 21, 30, 52, 128, 128, kept=0.24),
        _case("step_wan14b_480p", "step", 1, 40, 21, 30, 52, 128, 128, kept=0.24),
        # HunyuanVideo-shaped 720P with text blocks in front: the largest
        _case("step_hunyuan_720p", "step", 1, 24, 33, 45, 80, 128, 128, text=256, tau_lo=0.80, kept=0.19),
        # the dense warm-up steps
        _case("dense_wan1p3b_480p", "dense", 1, 12, 21, 30, 52, 128, 128, kept=1.0),
        # a step that reuses every mask, at the 15 % density asked for at 720P; folded softmax scale
        _case("attn_wan14b_720p_fold", "attn", 1, 40, 21, 45, 80, 128, 128, layout="bnhd", tau_lo=0.75,
              tau_hi=0.94, kept=0.15, fold=True),
        # the mask-refresh side alone: the second half of the benchmark's metric
        _case("refresh_wan14b_480p", "refresh", 1, 40, 21, 30, 52, 128, 128, kept=0.24),
        _case("refresh_hunyuan_720p", "refresh", 1, 24, 33, 45, 80, 128, 128, text=256, tau_lo=0.80, kept=0.19),
        # the alternative importance estimator and the selection from its scores
        _case("scores_wan14b_480p", "scores", 1, 40, 21, 30, 52, 128, 128, kept=0.29),
        # threshold calibration: one head's velocity over the 480P grid
        _case("ebc_480p", "ebc", 1, 1, 21, 30, 52, 128, 128, C=128),
    ]


def draw(rng):
    """One more case: tokens from a few hundred to the 720P clips, one head (a shard) to forty."""
    path = rng.choice(["step", "step", "step", "dense", "attn", "refresh", "refresh", "scores", "ebc"])
    D = rng.choice([128, 128, 128, 64])
    block = rng.choice([128, 128, 64])
    X = rng.randint(8, 80)
    Y = rng.randint(8, 45)
    if path == "ebc":
        return _case("", "ebc", 1, 1, rng.randint(3, 33), Y, X, 128, 128, C=rng.choice([16, 48, 64, 128]))
    T = max(1, int(round(math.exp(rng.uniform(0.0, math.log(33.0))))))
    text = rng.choice([0, 0, 0, block, 2 * block])
    while (T * Y * X + text + block - 1) // block > 1000:  # the mask ranks at most 1024 blocks per row
        T -= 1
    N = T * Y * X + text
    B = rng.choice([1, 1, 2])
    H = max(1, int(round(math.exp(rng.uniform(0.0, math.log(40.0))))))
    # (no more work than the largest listed case: its tokens squared times heads)
    cap = 24.0 * 119056.0 ** 2 * (0.2 if path == "dense" else 0.5)
    while B * H > 1 and B * H * float(N) ** 2 * D / 128.0 > cap:
        B, H = 1, max(1, H * B - 1)
    lo = rng.uniform(0.6, 0.9)
    return _case("", path, B, H, T, Y, X, D, block, text=text, layout=rng.choice(["bhnd", "bnhd"]),
                 tau_lo=lo, tau_hi=rng.uniform(lo, 0.98), kept=1.0 if path == "dense" else 0.25,
                 fold=path == "attn" and rng.random() < 0.5)


def _tokens(case):
    return case["text"] + case["T"] * case["Y"] * case["X"]


def _fields(case, seed, steps):
    """bf16 (q, k, v) of `steps` denoising steps, logical shape [B, H, N, D]."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(1_000_003 * seed + 17)
    B, H, D, T, Y, X, text = (case[n] for n in ("B", "H", "D", "T", "Y", "X", "text"))
    N = _tokens(case)
    n = torch.arange(T * Y * X, device=dev)
    pos = torch.stack([(n // (Y * X)) / T, ((n // X) % Y) / Y, (n % X) / X], dim=1)
    # frequencies over (t, y), the last of the four also along x; never constant over (t, y)
    freq = torch.stack([torch.randint(0, 4, (H, 4), generator=g, device=dev),
                        torch.randint(1, 5, (H, 4), generator=g, device=dev),
                        torch.randint(1, 4, (H, 4), generator=g, device=dev)], dim=2).float()
    freq[:, :3, 2] = 0.0
    phase = 2.0 * math.pi * torch.rand((H, 4), generator=g, device=dev)
    ell = 0.5 + 3.5 * torch.rand((H,), generator=g, device=dev)
    u = torch.randn((2, H, 4, D), generator=g, device=dev) / math.sqrt(D)  # Q and K share u[0]
    amp = math.sqrt(8.0 * math.sqrt(D) / 2.0)  # block logits span about 8
    # per-head offset of the second step: L1 size 4 delta for the heads that move
    jump = torch.zeros(H, device=dev)
    jump[torch.randperm(H, generator=g, device=dev)[:max(1, round(JUMP_SHARE * H))]] = 1.0
    size = DELTA * (0.01 + 3.99 * jump)
    dirs = (torch.randn((2, H, 4, 1), generator=g, device=dev) * u[0]).sum(2)  # in the field's span
    dirs = dirs / dirs.abs().sum(-1, keepdim=True)
    shape = (B, N, H, D) if case["layout"] == "bnhd" else (B, H, N, D)
    out = [[torch.empty(shape, dtype=torch.bfloat16, device=dev) for _ in range(3)] for _ in range(steps)]
    for h in range(H):
        s = torch.sin(2.0 * math.pi * (pos @ freq[h].T) / ell[h] + phase[h])
        fields = (s @ (amp * u[0, h]), s @ u[1, h])
        for b in range(B):
            for t in range(3):
                x = torch.empty((N, D), device=dev)
                x[:text] = 0.3 * torch.randn((text, D), generator=g, device=dev)
                x[text:] = fields[t == 2] + 0.1 * torch.randn((N - text, D), generator=g, device=dev)
                for i in range(steps):
                    if i and t < 2:
                        x = x + 0.5 * size[h] * dirs[t, h]
                    dst = out[i][t]
                    (dst[b, :, h] if case["layout"] == "bnhd" else dst[b, h]).copy_(x)
    if case["layout"] == "bnhd":
        out = [[x.transpose(1, 2) for x in step] for step in out]
    tau = case["tau_lo"] + (case["tau_hi"] - case["tau_lo"]) * torch.rand((H,), generator=g, device=dev)
    return [tuple(step) for step in out], tau


def prepare(case, seed):
    path = case["path"]
    if path == "ebc":
        g = torch.Generator(device="cuda").manual_seed(1_000_003 * seed + 29)
        shape = (case["C"], case["T"], case["Y"], case["X"])
        dense = torch.randn(shape, generator=g, device="cuda")
        # an error with some structure: a smooth part along every axis and noise
        err = 0.05 * torch.randn(shape, generator=g, device="cuda")
        err += 0.1 * (dense + dense.roll(1, 1) + dense.roll(1, 2) + dense.roll(1, 3)) / 4.0
        ws = torch.empty(heart.heart_ebc_workspace_bytes(*shape), dtype=torch.uint8, device="cuda")
        return {"path": path, "err": err, "dense": dense, "workspace": ws,
                "out": torch.empty(6, dtype=torch.float64, device="cuda")}
    inputs, tau = _fields(case, seed, 2 if path in ("step", "refresh") else 1)
    B, H, D, block = case["B"], case["H"], case["D"], case["block"]
    N = _tokens(case)
    Nb = (N + block - 1) // block
    nt = case["text"] // block
    q, k, v = inputs[0]
    state = {"path": path, "inputs": inputs, "turn": 0, "tau": tau, "block": block, "nt": nt}
    delta = torch.full((H,), DELTA, device="cuda")
    if path in ("step", "dense"):
        drv = TmrDriver(TmrConfig(B=B, H=H, N=N, D=D, block=block, tau=tau, delta=delta, gate=GATE,
                                  n_always_kv_blocks=nt, n_dense_q_blocks=nt), n_layers=1, n_branches=1)
        state.update(driver=drv, out=torch.empty_like(q))
        if path == "step":  # the first sparse step, which refreshes every head, is over
            drv.attention(0, 0, drv.cfg.dense_steps, q, k, v, out=state["out"])
        return state
    f32 = dict(dtype=torch.float32, device="cuda")
    lists = dict(mask=torch.zeros((B, H, Nb, Nb), dtype=torch.uint8, device="cuda"),
                 kept_idx=torch.zeros((B, H, Nb, Nb), dtype=torch.int32, device="cuda"),
                 kept_count=torch.zeros((B, H, Nb), dtype=torch.int32, device="cuda"))
    state["lists"] = lists
    if path == "attn":
        qblk, kblk, _, _ = heart.heart_pool_qk(q, k, block)
        heart.heart_mask_topp(qblk, kblk, tau, n_always_kv_blocks=nt, n_dense_q_blocks=nt, **lists)
        state.update(out=torch.empty_like(q), lse=torch.empty((B, H, N), **f32),
                     flags=heart.HEART_ATTN_FOLD_SCALE if case["fold"] else 0,
                     workspace=torch.empty(heart.heart_attn_workspace_bytes(q, block), dtype=torch.uint8,
                                           device="cuda"))
    elif path == "scores":
        state.update(scores=torch.empty((B, H, Nb, Nb), **f32), workspace=torch.empty(
            heart.heart_scores_antidiag_workspace_bytes(q, block, block // 8), dtype=torch.uint8, device="cuda"))
    else:
        state["pool"] = dict(qblk=torch.empty((B, H, Nb, D), **f32), kblk=torch.empty((B, H, Nb, D), **f32),
                             qmean=torch.empty((B, H, D), **f32), kmean=torch.empty((B, H, D), **f32),
                             drift=torch.empty((B, H), **f32),
                             refresh=torch.empty((B, H), dtype=torch.uint8, device="cuda"))
        state["anchor"] = (torch.zeros((B, H, D), **f32), torch.zeros((B, H, D), **f32),
                           torch.zeros((B, H), dtype=torch.uint8, device="cuda"), delta)
        state["tickets"] = torch.zeros(heart.heart_pool_drift_workspace_bytes(B, H), dtype=torch.uint8,
                                       device="cuda")
        state["topp_ws"] = None
        if Nb > SLICED_SCORES_MIN_NB:
            state["topp_ws"] = torch.empty(heart.heart_mask_topp_workspace_bytes(B, H, Nb, D),
                                           dtype=torch.uint8, device="cuda")
        _refresh(state, q, k)  # the first sparse step is over
    return state


def _refresh(state, q, k):
    pool = state["pool"]
    heart.heart_pool_drift(q, k, state["block"], *state["anchor"], state["tickets"], GATE[0], GATE[1], True,
                           **pool)
    heart.heart_mask_topp(pool["qblk"], pool["kblk"], state["tau"], refresh=pool["refresh"],
                          n_always_kv_blocks=state["nt"], n_dense_q_blocks=state["nt"],
                          workspace=state["topp_ws"], **state["lists"])


def run(state):
    path = state["path"]
    if path == "ebc":
        return heart.heart_ebc_band_error(state["err"], state["dense"], workspace=state["workspace"],
                                          out=state["out"])
    state["turn"] = (state["turn"] + 1) % len(state["inputs"])
    q, k, v = state["inputs"][state["turn"]]
    if path in ("step", "dense"):
        drv = state["driver"]
        drv.attention(0, 0, drv.cfg.dense_steps if path == "step" else 0, q, k, v, out=state["out"])
        if path == "dense":
            return state["out"]
        st = drv.states[(0, 0)]
        return {"out": state["out"], "drift": st.drift, "refresh": st.refresh, "qanchor": st.qanchor,
                "kanchor": st.kanchor, "mask": st.mask, "kept_idx": st.kept_idx, "kept_count": st.kept_count}
    lists = state["lists"]
    if path == "attn":
        heart.heart_block_sparse_attn_flags(q, k, v, state["block"], lists["kept_idx"], lists["kept_count"],
                                            state["flags"], out=state["out"], lse=state["lse"],
                                            workspace=state["workspace"])
        return state["out"], state["lse"]
    if path == "scores":
        heart.heart_scores_antidiag(q, k, state["block"], state["block"] // 8, scores=state["scores"],
                                    workspace=state["workspace"])
        heart.heart_mask_topp(None, None, state["tau"], scores_in=state["scores"],
                              n_always_kv_blocks=state["nt"], n_dense_q_blocks=state["nt"], **lists)
        return {"scores": state["scores"], **lists}
    _refresh(state, q, k)
    return {**state["pool"], **lists}


def work(case):
    """Each input read once, each output written once; the products the method asks for."""
    path = case["path"]
    if path == "ebc":
        n = case["T"] * case["Y"] * case["X"]
        total = case["C"] * n
        # (a real transform of the error, its band energies, the energy of the reference)
        return {"bytes": 2.0 * 4 * total, "flops": total * (2.5 * math.log2(max(2, n)) + 4.0)}
    B, H, D, block = case["B"], case["H"], case["D"], case["block"]
    N = _tokens(case)
    Nb = (N + block - 1) // block
    tensor = 2.0 * B * H * N * D                  # bytes of one bf16 tensor
    attn = 4.0 * D * B * H * float(N) ** 2 * case["kept"]
    lists = B * H * (Nb * Nb * (1.0 + 4.0 * case["kept"]) + 4.0 * Nb)  # mask, kept lists, counts
    pairs = 2.0 * D * B * H * float(Nb) ** 2      # block scores
    if path == "dense":
        return {"bytes": 4 * tensor, "flops": attn}
    if path == "attn":
        return {"bytes": 4 * tensor + lists - B * H * Nb * Nb + 4.0 * B * H * N, "flops": attn}
    if path == "scores":
        M = math.ceil(N / (block // 8))
        return {"bytes": 2 * tensor + lists + 4.0 * B * H * Nb * Nb,
                "flops": 2.0 * float(M) ** 2 * (block // 8) * D * B * H}
    blocks = 8.0 * B * H * (Nb + 1) * D           # block and token means of Q and K
    if path == "refresh":
        return {"bytes": 2 * tensor + blocks + JUMP_SHARE * lists,
                "flops": 2.0 * B * H * N * D + JUMP_SHARE * pairs}
    return {"bytes": 4 * tensor + JUMP_SHARE * lists, "flops": attn + 2.0 * B * H * N * D + JUMP_SHARE * pairs}


def tolerance(case):
    """About four times what another correct implementation at the same precision differs by, measured
    at the listed sizes: attention against its other softmax-scale path (rel 1.3e-3, max 1.35e-2, one
    bf16 rounding of the output), block means against 64-bit sums (max 1.2e-7) with the lists that follow
    from them (no entry differs; one row at its threshold in ten thousand may), scores against 64-bit
    products (rel 4.6e-7, max 5e-6), band energies against a 64-bit FFT (rel 2e-16; sums of some
    million terms in another order)."""
    path = case["path"]
    if path == "ebc":
        return {"rel": 1e-12, "max": 1e-12}
    if path in ("dense", "attn"):
        return {"rel": 5e-3, "max": 0.055}
    if path == "scores":
        return {"rel": 2e-6, "max": 2e-5, "differ": 1e-4}
    if path == "refresh":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-4}
    return {"rel": 5e-3, "max": 0.055, "differ": 1e-4}
