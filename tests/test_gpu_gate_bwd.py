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


@pytest.mark.parametrize("S", [16, 100, 4096, 5000, 70001])
def test_bias_gradient_rounding(S):
    """The bias gradient of up to 16 experts: fp32 sums over quarters of a token chunk, added up in fp64.  At most
    chunk / 4 + 2 fp32 additions reach a term, each off by at most 2^-24 of a sum no larger than the chunk's sum of
    magnitudes, and the result is rounded once: |error| <= (chunk / 4 + 3) 2^-24 sum |dlogits|.  One large term per 16
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
    chunk = -(-(-(-S // 256)) // 16) * 16
    bound = (chunk / 4 + 3) * 2.0 ** -24 * np.abs(l64).sum(axis=0)
    assert (np.abs(to_host(db) - l64.sum(axis=0)) <= bound).all()
