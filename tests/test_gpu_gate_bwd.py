"""GPU parity: backward of the gate against the CPU checker."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2407_00599_amd import api, synth
from util import DEV, ROWS, assert_close, to_dev, to_host, rel_err, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,M,E,k,norm,dtype,acc", [
    (1, 8, 1, 1, 0, "f32", 0), (256, 64, 4, 1, 0, "f32", 1), (300, 72, 8, 2, 1, "f32", 1), (1000, 1024, 8, 2, 1, "bf16", 1),
    (777, 264, 16, 4, 0, "bf16", 0), (513, 128, 64, 2, 1, "bf16", 1), (400, 200, 100, 8, 0, "f32", 0),
    (2100, 2048, 17, 3, 1, "bf16", 1), (64, 64, 256, 8, 1, "f32", 1),
    # bf16, at most 8 experts, thousands of tokens (blocks of the fused kernel walk several 16-token stages): ragged
    # token and column tails, fewer than 8 experts, both weight normalisations, more than 65536 tokens
    (2048, 256, 8, 1, 0, "bf16", 1), (2049, 264, 8, 2, 1, "bf16", 1), (4099, 1032, 5, 2, 0, "bf16", 0),
    (3000, 520, 1, 1, 0, "bf16", 1), (70001, 72, 8, 2, 1, "bf16", 1),
    # edges of the fused kernel's waves and chunks (4 tokens a stage, 16 a block, 256 dlogits rows at a time), of its 256
    # columns, and of the matrix-core kernels' 32 tokens, 128 columns and 8, 32, 64, 128 experts
    (15, 256, 16, 2, 1, "bf16", 1), (17, 264, 13, 3, 0, "f32", 1), (4097, 248, 8, 1, 0, "f32", 0), (70001, 8, 16, 2, 1, "f32", 1),
    (31, 136, 24, 2, 0, "bf16", 1), (33, 120, 32, 4, 1, "f32", 0), (65, 128, 33, 1, 0, "bf16", 1), (127, 8, 64, 6, 1, "bf16", 1),
    (4097, 520, 65, 2, 0, "f32", 1), (129, 264, 128, 8, 1, "bf16", 0), (300, 24, 129, 3, 0, "bf16", 1),
])
def test_gate_bwd(S, M, E, k, norm, dtype, acc):
    rng = np.random.default_rng(S + E)
    x = synth.store(rng.standard_normal((S, M)).astype(np.float32), dtype)
    Wg = (rng.standard_normal((M, E)) * 0.1).astype(np.float32)
    logits = synth.synthetic_logits(S, E, seed=S)
    idx = O.topk_select(logits, k)
    w = O.combine_weights(logits, idx, bool(norm)).astype(np.float32)
    dw = rng.standard_normal((S, k)).astype(np.float32)
    dx0 = synth.store(rng.standard_normal((S, M)).astype(np.float32), dtype)
    tdt = torch_dtype(dtype)
    dl = torch.empty(S, E, device=DEV); dWg = torch.empty(M, E, device=DEV); db = torch.empty(E, device=DEV)
    dx = to_dev(dx0).clone()
    # a workspace full of 0xFF bytes (NaN as bf16 or fp32): nothing may be read from it that the call has not written
    ws = torch.full((api.moe_gate_bwd_workspace_bytes(S, M, E),), 255, dtype=torch.uint8, device=DEV)
    api.moe_gate_bwd(to_dev(dw), to_dev(w), to_dev(idx), to_dev(logits), to_dev(x), to_dev(Wg), S, M, E, k, norm,
                     dl, dWg, db, dx, acc, ws)
    torch.cuda.synchronize()
    rdl, rdWg, rdb, rdx = O.gate_bwd(dw, logits, idx, bool(norm), x.val, Wg)
    assert rel_err(to_host(dl), rdl) <= 1e-5
    assert rel_err(to_host(dWg), rdWg) <= 1e-5
    assert rel_err(to_host(db), rdb) <= 1e-5
    ref_dx = rdx + (dx0.val if acc else 0.0)
    assert rel_err(to_host(dx), ref_dx) <= (1e-5 if dtype == "f32" else 4e-3)
    assert_close(to_host(dWg), rdWg, 1e-5, "dWg")
    assert_close(to_host(db), rdb, 1e-5, "dbias")
    assert_close(to_host(dx), ref_dx, 1e-5 if dtype == "f32" else 4e-3, "dx", ROWS)
    if k == 1 and norm:
        assert np.all(to_host(dl) == 0)


# the slab of Wg in 16-byte pieces (4 | E) that end within a block's 256 columns or behind them, and element by element; stages that are
# requested before the dlogits rows of the next 256 tokens exist.  (norm_topk in fp32 with an old dx: dl[e_j] = w_j (dw_j - sum w dw) is
# off by up to (k + 2) 2^-24 max|dw| times w_j where it cancels, and a row of dx consists of nothing else without one.)
@pytest.mark.parametrize("S,M,E,k,norm,dtype,acc", [
    (19, 40, 12, 3, 1, "bf16", 0), (300, 280, 12, 8, 1, "f32", 1), (66003, 32, 12, 2, 0, "bf16", 1), (66003, 24, 6, 2, 1, "f32", 1),
    (2100, 264, 10, 4, 0, "bf16", 1),
    # numbers of experts that are no multiple of 4: the slab in threes of values, whole and ragged columns
    (50, 256, 2, 1, 0, "f32", 0), (40, 264, 3, 2, 1, "bf16", 1), (40, 8, 7, 3, 1, "f32", 1), (50, 520, 9, 2, 1, "bf16", 0), (40, 256, 11, 4, 0, "f32", 1),
    (30, 504, 15, 8, 1, "f32", 0),
])
def test_gate_bwd_slab_and_stages(S, M, E, k, norm, dtype, acc):
    test_gate_bwd(S, M, E, k, norm, dtype, acc)


@pytest.mark.parametrize("S", [16, 100, 2048, 4096, 5000, 70001])
def test_bias_gradient_rounding(S):
    """The bias gradient of up to 16 experts: fp32 sums over quarters of a token chunk, added up in fp64 and rounded.  At most
    chunk / 4 fp32 additions and that rounding reach a term, each off by at most 2^-24 of a sum no larger than the chunk's
    sum of magnitudes, and the result is rounded once: |error| <= (chunk / 4 + 2) 2^-24 sum |dlogits|.  One large term per 16
    tokens among terms that vanish next to it, so that one long chain over 16 tokens would miss the bound."""
    M, E, k = 8, 8, 2
    g = np.where(np.arange(S) % 16 == 0, 4.0, 4.0 * 2.0 ** -25)
    dw = np.stack([g, np.zeros(S)], 1).astype(np.float32)                  # dl[t, 0] = 0.25 (dw0 - dw1) = -dl[t, 1]
    idx = np.tile(np.array([0, 1], np.int32), (S, 1))
    w = np.full((S, k), 0.5, np.float32)
    dl = torch.empty(S, E, device=DEV); dWg = torch.empty(M, E, device=DEV); db = torch.empty(E, device=DEV)
    dx = torch.empty(S, M, device=DEV)
    ws = torch.full((api.moe_gate_bwd_workspace_bytes(S, M, E),), 255, dtype=torch.uint8, device=DEV)
    api.moe_gate_bwd(to_dev(dw), to_dev(w), to_dev(idx), torch.zeros(S, E, device=DEV), torch.zeros(S, M, device=DEV),
                     torch.zeros(M, E, device=DEV), S, M, E, k, 1, dl, dWg, db, dx, 0, ws)
    torch.cuda.synchronize()
    l64 = to_host(dl)
    assert np.array_equal(l64[:, 0], g / 4) and np.array_equal(l64[:, 1], -g / 4)
    chunk = -(-(-(-S // (64 if S <= 2048 else 256))) // 16) * 16
    bound = (chunk / 4 + 2) * 2.0 ** -24 * np.abs(l64).sum(axis=0)
    assert (np.abs(to_host(db) - l64.sum(axis=0)) <= bound).all()


@pytest.mark.parametrize("S,M,E,k,norm,dtype", [(1003, 520, 12, 3, 1, "bf16"), (1000, 264, 16, 2, 1, "f32"), (2048, 256, 8, 2, 1, "bf16"),
                                                (8, 2048, 8, 2, 1, "f32"), (1032, 264, 8, 2, 1, "f32"), (4096, 264, 8, 2, 1, "bf16"), (5000, 264, 13, 2, 0, "f32")])
def test_weight_gradient_rounding(S, M, E, k, norm, dtype):
    """The weight gradient of up to 16 experts is no farther from the exact sums than fp32 chains over chunks of 8 tokens (more
    from 2049 tokens on: at most 256 chunks), added up in fp64 and rounded.  Chains of equal length over other tokens have
    equal errors on average; over N outputs the two norms of N independent errors then differ by 1 / sqrt(N) of
    themselves in the standard deviation, of which four are allowed."""
    rng = np.random.default_rng(S * 3 + E)
    x = synth.store(rng.standard_normal((S, M)).astype(np.float32), dtype)
    logits = synth.synthetic_logits(S, E, seed=S)
    idx = O.topk_select(logits, k)
    w = O.combine_weights(logits, idx, bool(norm)).astype(np.float32)
    dw = rng.standard_normal((S, k)).astype(np.float32)
    dl = torch.empty(S, E, device=DEV); dWg = torch.empty(M, E, device=DEV); db = torch.empty(E, device=DEV)
    dx = torch.empty(S, M, dtype=torch_dtype(dtype), device=DEV)
    ws = torch.full((api.moe_gate_bwd_workspace_bytes(S, M, E),), 255, dtype=torch.uint8, device=DEV)
    api.moe_gate_bwd(to_dev(dw), to_dev(w), to_dev(idx), to_dev(logits), to_dev(x), torch.zeros(M, E, device=DEV), S, M, E, k, norm,
                     dl, dWg, db, dx, 0, ws)
    torch.cuda.synchronize()
    x64, l64 = x.val.astype(np.float64), to_host(dl)
    exact = x64.T @ l64
    chunk = max(8, -(-(-(-S // 256)) // 8) * 8)
    chained = np.zeros((M, E))
    for t0 in range(0, S, chunk):
        acc = np.zeros((M, E), np.float32)
        for t in range(t0, min(S, t0 + chunk)):
            acc = (acc + x64[t][:, None] * l64[t][None, :]).astype(np.float32)      # fused multiply-add: one rounding
        chained += acc
    err = lambda a: np.linalg.norm(a - exact)      # noqa: E731
    assert err(to_host(dWg)) <= (1 + 4 / np.sqrt(M * E)) * err(chained.astype(np.float32).astype(np.float64))

    # infinities stay infinities
    t, e = S // 2, int(idx[S // 2, 0])
    xi = to_dev(x).clone()
    xi[t, 3] = float("inf")
    api.moe_gate_bwd(to_dev(dw), to_dev(w), to_dev(idx), to_dev(logits), xi, torch.zeros(M, E, device=DEV), S, M, E, k, norm,
                     dl, dWg, db, dx, 0, ws)
    torch.cuda.synchronize()
    assert to_host(dWg)[3, e] == np.inf * np.sign(l64[t, e]) and np.isfinite(np.delete(to_host(dWg), 3, axis=0)).all()
