"""GPU parity: ESP-sharded expert FFN forward and backward against the CPU checker.

Moderate shapes are compared element by element (several tiles, ragged tails, n_src chunks,
ESP slices, both workgroup tiles); the two largest benchmark shapes are run at full size in the
launch configuration the benchmark uses and checked on sampled rows and hidden units."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2407_00599_amd import api, synth
from util import DEV, TOL, ROWS, EXPERT, to_dev, to_host, rel_err, assert_close, torch_dtype

pytestmark = pytest.mark.gpu


def gpu_ffn(X, dY, W1, W2, n_src, G, C, M, H, esp_idx, n_esp, tdt, row_counts=None, tile=0, ws_bytes=None):
    """Every output but the full-size weight gradients (3.0) starts as NaN, and so does the scratch memory: a row that no
    workgroup stores, or a read of one that nobody writes, shows."""
    Hl = H // n_esp
    dt = api.MOE_BF16 if tdt == torch.bfloat16 else api.MOE_F32
    new = lambda *s, v=float("nan"): torch.full(s, v, dtype=tdt, device=DEV)      # noqa: E731
    Z, A = new(n_src, G, C, Hl), new(n_src, G, C, Hl)
    Y, dX = new(n_src, G, C, M), new(n_src, G, C, M)
    dW1, dW2 = new(G, M, H, v=3.0), new(G, H, M, v=3.0)
    if ws_bytes is None:
        ws_bytes = api.moe_ffn_workspace_bytes(dt, n_src, G, C, M, H, n_esp)
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device=DEV)
    api.moe_expert_ffn_fwd(X, W1, W2, n_src, G, C, M, H, esp_idx, n_esp, Z, A, Y, row_counts, tile)
    api.moe_expert_ffn_bwd(dY, X, Z, A, W1, W2, n_src, G, C, M, H, esp_idx, n_esp, dX, dW1, dW2, ws, row_counts, tile)
    torch.cuda.synchronize()
    return Z, A, Y, dX, dW1, dW2


SMALL, T256, T192 = api.MOE_TILE_SMALL, api.MOE_TILE_256, api.MOE_TILE_192
CASES = [
    # n_src, G, C, M, H, n_esp, esp_idx, dtype, tile hint (0 = auto)
    (1, 4, 77, 64, 128, 1, 0, "f32", 0),
    (3, 2, 100, 72, 256, 2, 1, "f32", 0),
    (2, 1, 33, 200, 104, 1, 0, "f32", 0),
    (1, 2, 130, 128, 256, 1, 0, "bf16", SMALL),
    (3, 2, 150, 256, 512, 2, 1, "bf16", SMALL),
    (1, 2, 300, 512, 768, 1, 0, "bf16", T256),
    (2, 3, 200, 264, 1040, 2, 0, "bf16", T256),
    (3, 2, 77, 136, 520, 1, 0, "bf16", T256),
    (2, 2, 150, 256, 512, 2, 1, "bf16", T256),
    (1, 2, 300, 512, 768, 1, 0, "bf16", T192),
    (2, 3, 230, 264, 1040, 2, 0, "bf16", T192),
    (3, 2, 77, 136, 520, 1, 0, "bf16", T192),
    (4, 2, 70, 136, 520, 1, 0, "bf16", SMALL),
    (1, 1, 1, 8, 8, 1, 0, "bf16", SMALL),
    (5, 1, 64, 1024, 64, 4, 3, "bf16", 0),
    (4, 4, 256, 768, 3072, 1, 0, "bf16", 0),      # the rank-shaped FFN of workload "mp4_ep": n_src = 4, G = 4, C = 256
]


@pytest.mark.parametrize("n_src,G,C,M,H,n_esp,esp_idx,dtype,tile", CASES)
def test_ffn_fwd_bwd_elementwise(n_src, G, C, M, H, n_esp, esp_idx, dtype, tile):
    rng = np.random.default_rng(n_src * 1000 + C)
    tdt = torch_dtype(dtype)
    Xn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    dYn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    for s in range(n_src):                       # capacity padding: zero tails
        for g in range(G):
            occ = int(rng.integers(0, C + 1))
            Xn[s, g, occ:] = 0; dYn[s, g, occ:] = 0
    X, dY = synth.store(Xn, dtype), synth.store(dYn, dtype)
    W1 = synth.store((rng.standard_normal((G, M, H)) / np.sqrt(M)).astype(np.float32), dtype)
    W2 = synth.store((rng.standard_normal((G, H, M)) / np.sqrt(H)).astype(np.float32), dtype)
    Z, A, Y, dX, dW1, dW2 = gpu_ffn(to_dev(X), to_dev(dY), to_dev(W1), to_dev(W2), n_src, G, C, M, H, esp_idx, n_esp, tdt,
                                    tile=tile)
    rZ, rY = O.expert_ffn_fwd(X.val, W1.val, W2.val, esp_idx, n_esp)
    rdX, rdW1, rdW2 = O.expert_ffn_bwd(dY.val, X.val, W1.val, W2.val, esp_idx, n_esp)
    tol = TOL[dtype]
    Hl = H // n_esp; hs = slice(esp_idx * Hl, (esp_idx + 1) * Hl)
    assert_close(to_host(Z), rZ, tol, "Z", ROWS)
    assert_close(to_host(A), O.gelu(rZ), tol, "A", ROWS)
    assert_close(to_host(Y), rY, tol, "Y", ROWS)
    assert_close(to_host(dX), rdX, tol, "dX", ROWS)
    hW1, hW2 = to_host(dW1), to_host(dW2)
    assert_close(hW1[:, :, hs], rdW1, tol, "dW1", EXPERT)
    assert_close(hW2[:, hs, :], rdW2, tol, "dW2", EXPERT)
    # the other shards' columns / rows of the full gradient tensors are not touched
    mask = np.ones(H, bool); mask[hs] = False
    assert np.all(hW1[:, :, mask] == 3.0) and np.all(hW2[:, mask, :] == 3.0)
    # padding rows produce exact zeros
    zero_rows = ~X.val.any(axis=-1)
    assert np.all(to_host(Y)[zero_rows] == 0.0)


@pytest.mark.parametrize("n_src,G,C,M,H,occ,tile", [
    (1, 3, 700, 256, 512, [[0, 130, 700]], 0),          # an empty expert, one short, one full (auto tiles)
    (1, 3, 700, 256, 512, [[1, 257, 900]], T256),       # a demand count above the capacity
    (1, 2, 600, 264, 520, [[193, 384]], T192),          # 192-row tiles, counts at tile edges
    (3, 2, 300, 256, 512, [[0, 300], [40, 0], [299, 1]], 0),   # several source chunks
    (2, 1, 150, 128, 256, [[10, ], [149, ]], SMALL),    # small problem: the register-staged kernel ignores the counts
    # weight gradients whose reductions are cut into parts: one chunk, half and all of it occupied; a chunk almost empty; several
    (1, 2, 1700, 136, 264, [[850, 1700]], 0),
    (1, 1, 3300, 72, 136, [[1001]], 0),
    (2, 2, 1100, 136, 264, [[1100, 3], [65, 0]], 0),
    (3, 1, 1100, 264, 520, [[0], [1100], [300]], 0),
])
def test_row_counts_change_nothing(n_src, G, C, M, H, occ, tile):
    """Telling the FFN which rows are capacity padding must not change any result (only the time)."""
    rng = np.random.default_rng(99)
    Xn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    dYn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    for s in range(n_src):
        for g in range(G):
            Xn[s, g, occ[s][g]:] = 0; dYn[s, g, occ[s][g]:] = 0
    X, dY = to_dev(synth.store(Xn, "bf16")), to_dev(synth.store(dYn, "bf16"))
    W1 = to_dev(synth.store((rng.standard_normal((G, M, H)) / np.sqrt(M)).astype(np.float32), "bf16"))
    W2 = to_dev(synth.store((rng.standard_normal((G, H, M)) / np.sqrt(H)).astype(np.float32), "bf16"))
    cnt = torch.tensor(occ, dtype=torch.int32, device=DEV)
    ref = gpu_ffn(X, dY, W1, W2, n_src, G, C, M, H, 0, 1, torch.bfloat16, tile=tile)
    got = gpu_ffn(X, dY, W1, W2, n_src, G, C, M, H, 0, 1, torch.bfloat16, cnt, tile=tile)
    for name, a, b in zip(("Z", "A", "Y", "dX", "dW1", "dW2"), ref, got):
        assert torch.equal(a.float(), b.float()), name      # == on values: -0 and +0 count as equal
    assert not (ref[2][X.abs().sum(-1) == 0] != 0).any()


def _device_inputs(cfg, C, seed):
    """Rank-shaped inputs drawn on the device (same distributions as the host generator)."""
    gen = torch.Generator(device=DEV); gen.manual_seed(synth.BASE_SEED + seed)
    tdt = torch.bfloat16
    rn = lambda *s, sig=1.0: (torch.randn(*s, generator=gen, device=DEV, dtype=torch.float32) * sig).to(tdt)
    X = rn(cfg.n_src, cfg.G, C, cfg.M); dY = rn(cfg.n_src, cfg.G, C, cfg.M)
    occ = torch.randint(C // 2, C + 1, (cfg.n_src, cfg.G), generator=gen, device=DEV)
    pad = torch.arange(C, device=DEV)[None, None, :] >= occ[:, :, None]
    X[pad] = 0; dY[pad] = 0
    W1 = torch.empty(cfg.G, cfg.M, cfg.H, dtype=tdt, device=DEV); W2 = torch.empty(cfg.G, cfg.H, cfg.M, dtype=tdt, device=DEV)
    for g in range(cfg.G):
        W1[g] = rn(cfg.M, cfg.H, sig=cfg.sigma_w); W2[g] = rn(cfg.H, cfg.M, sig=cfg.sigma_w)
    return X, dY, W1, W2


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name", ["esp4", "large"])
def test_ffn_full_size_sampled(name):
    cfg = synth.CONFIGS[name]
    C = O.capacity(cfg.S, cfg.E, cfg.k, cfg.f)
    n_src, G, M, H, Hl = cfg.n_src, cfg.G, cfg.M, cfg.H, cfg.H_local
    X, dY, W1, W2 = _device_inputs(cfg, C, cfg.cfg_id)
    Z, A, Y, dX, dW1, dW2 = gpu_ffn(X, dY, W1, W2, n_src, G, C, M, H, cfg.esp_idx, cfg.n_esp, torch.bfloat16)
    hs = slice(cfg.esp_idx * Hl, (cfg.esp_idx + 1) * Hl)
    rng = np.random.default_rng(cfg.cfg_id)
    tol = TOL["bf16"]
    for g in (0, G - 1):
        w1s = to_host(W1[g][:, hs]); w2s = to_host(W2[g][hs, :])
        pick = [(0, 0), (n_src - 1, C - 1), (n_src // 2, C // 2)] + \
               [(int(rng.integers(n_src)), int(rng.integers(C))) for _ in range(13)]
        ss = torch.tensor([p[0] for p in pick], device=DEV); cc = torch.tensor([p[1] for p in pick], device=DEV)
        z, y, dx = O.expert_ffn_rows(to_host(X[ss, g, cc]), to_host(dY[ss, g, cc]), w1s, w2s)
        assert_close(to_host(Z[ss, g, cc]), z, tol, "Z", ROWS)
        assert_close(to_host(A[ss, g, cc]), O.gelu(z), tol, "A", ROWS)
        assert_close(to_host(Y[ss, g, cc]), y, tol, "Y", ROWS)
        assert_close(to_host(dX[ss, g, cc]), dx, tol, "dX", ROWS)
        Xg = to_host(X[:, g].reshape(n_src * C, M)); dYg = to_host(dY[:, g].reshape(n_src * C, M))
        for h in [0, Hl - 1] + [int(rng.integers(Hl)) for _ in range(3)]:
            c1, r2 = O.expert_ffn_hidden_unit(Xg, dYg, w1s[:, h], w2s[h, :])
            assert_close(to_host(dW1[g, :, hs.start + h]), c1, tol, "dW1")
            assert_close(to_host(dW2[g, hs.start + h, :]), r2, tol, "dW2")
        del Xg, dYg
    # rows that are capacity padding stay exactly zero, at any size
    zero_rows = ~(X != 0).any(dim=-1)
    assert zero_rows.any()
    assert not (Y[zero_rows] != 0).any()
