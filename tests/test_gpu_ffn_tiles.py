"""GPU parity of the expert FFN over the tiles that the plan picks by itself (few to some hundred rows per
expert, ragged in every dimension) and over the compacted row order: several source chunks with row counts,
more than 64 of them, more than 16 and more than 64 experts, empty and overfull chunks."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2407_00599_amd import api, synth
from test_gpu_ffn import gpu_ffn
from util import DEV, TOL, ROWS, EXPERT, to_dev, to_host, assert_close, torch_dtype

pytestmark = pytest.mark.gpu

CASES = [
    # n_src, G, C, M, H
    (1, 8, 20, 264, 520),      # fewer rows than the smallest tile
    (1, 3, 33, 1024, 2056),    # one row past it, long reductions
    (1, 4, 64, 512, 1032),
    (1, 12, 100, 520, 264),
    (2, 6, 150, 200, 1544),
    (6, 3, 130, 1032, 72),
    (1, 6, 129, 640, 1288),
    (3, 20, 40, 72, 136),      # more than 16 experts
    (1, 80, 6, 64, 64),        # more than 64 experts
    (70, 2, 9, 136, 264),      # more than 64 chunks
]
CASES_F32 = [
    (1, 8, 200, 72, 2056),     # enough tiles for 64 x 64 in the wide GEMMs, 32 x 32 in the narrow ones
    (2, 6, 150, 200, 1544),
    (1, 3, 33, 40, 72),
    (3, 20, 40, 72, 136),
    (70, 2, 9, 136, 264),
]


@pytest.mark.parametrize("n_src,G,C,M,H,dtype", [c + ("bf16",) for c in CASES] + [c + ("f32",) for c in CASES_F32])
def test_auto_tiles_and_compacted_rows(n_src, G, C, M, H, dtype):
    rng = np.random.default_rng(n_src * 7919 + C)
    occ = rng.integers(-C // 2, C + 2, size=(n_src, G)).clip(0)          # a third of the chunks empty, some at or above C
    Xn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    dYn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    for s in range(n_src):
        for g in range(G):
            Xn[s, g, occ[s, g]:] = 0; dYn[s, g, occ[s, g]:] = 0
    X, dY = synth.store(Xn, dtype), synth.store(dYn, dtype)
    W1 = synth.store((rng.standard_normal((G, M, H)) / np.sqrt(M)).astype(np.float32), dtype)
    W2 = synth.store((rng.standard_normal((G, H, M)) / np.sqrt(H)).astype(np.float32), dtype)
    cnt = torch.tensor(occ.astype(np.int32), device=DEV)
    args = [to_dev(t) for t in (X, dY, W1, W2)]
    got = gpu_ffn(*args, n_src, G, C, M, H, 0, 1, torch_dtype(dtype), cnt)
    rZ, rY = O.expert_ffn_fwd(X.val, W1.val, W2.val, 0, 1)
    rdX, rdW1, rdW2 = O.expert_ffn_bwd(dY.val, X.val, W1.val, W2.val, 0, 1)
    tol = TOL[dtype]
    for name, t, ref, group in (("Z", got[0], rZ, ROWS), ("A", got[1], O.gelu(rZ), ROWS), ("Y", got[2], rY, ROWS),
                                ("dX", got[3], rdX, ROWS), ("dW1", got[4], rdW1, EXPERT), ("dW2", got[5], rdW2, EXPERT)):
        assert_close(to_host(t), ref, tol, name, group)
    pad = ~X.val.any(axis=-1)
    for t in got[:4]:
        assert np.all(to_host(t)[pad] == 0.0)
    for _ in range(4):         # the pipeline's requests race with nothing: every run gives the same bits
        for a, b in zip(got, gpu_ffn(*args, n_src, G, C, M, H, 0, 1, torch_dtype(dtype), cnt)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("tile", [api.MOE_TILE_SMALL, api.MOE_TILE_256, api.MOE_TILE_192])
def test_fp32_ignores_the_tile_hint(tile):
    """The row counts hold whatever the hint: rows behind them, here full of values, are taken as padding."""
    n_src, G, C, M, H = 2, 3, 45, 72, 136
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    new = lambda *s: torch.randn(*s, generator=gen, device=DEV)      # noqa: E731
    X, dY, W1, W2 = new(n_src, G, C, M), new(n_src, G, C, M), new(G, M, H), new(G, H, M)
    cnt = torch.tensor([[0, 45, 7], [40, 1, 33]], dtype=torch.int32, device=DEV)
    run = lambda t: gpu_ffn(X, dY, W1, W2, n_src, G, C, M, H, 0, 1, torch.float32, cnt, t)      # noqa: E731
    for a, b in zip(run(api.MOE_TILE_AUTO), run(tile)):
        assert torch.equal(a, b)


def check_ffn(rng, n_src, G, C, M, H, dtype, tile, occ):
    """Forward and backward against the CPU checker; occ [n_src, G] = row counts that are passed, None = none are."""
    Xn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    dYn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    if occ is not None:
        pad = np.arange(C)[None, None, :] >= occ[:, :, None]
        Xn[pad] = 0; dYn[pad] = 0
    X, dY = synth.store(Xn, dtype), synth.store(dYn, dtype)
    W1 = synth.store((rng.standard_normal((G, M, H)) / np.sqrt(M)).astype(np.float32), dtype)
    W2 = synth.store((rng.standard_normal((G, H, M)) / np.sqrt(H)).astype(np.float32), dtype)
    cnt = None if occ is None else torch.tensor(occ.astype(np.int32), device=DEV)
    got = gpu_ffn(*(to_dev(t) for t in (X, dY, W1, W2)), n_src, G, C, M, H, 0, 1, torch_dtype(dtype), cnt, tile)
    rZ, rY = O.expert_ffn_fwd(X.val, W1.val, W2.val, 0, 1)
    rdX, rdW1, rdW2 = O.expert_ffn_bwd(dY.val, X.val, W1.val, W2.val, 0, 1)
    for name, t, ref, group in (("Z", got[0], rZ, ROWS), ("A", got[1], O.gelu(rZ), ROWS), ("Y", got[2], rY, ROWS),
                                ("dX", got[3], rdX, ROWS), ("dW1", got[4], rdW1, EXPERT), ("dW2", got[5], rdW2, EXPERT)):
        assert_close(to_host(t), ref, TOL[dtype], name, group)


@pytest.mark.parametrize("n_src,G,C,M,H,dtype,tile,counted", [
    (1, 2, 2200, 64, 2056, "bf16", api.MOE_TILE_SMALL, False),     # contiguous ranges: over 32 tiles per XCD, over 16 row tiles
    (1, 2, 2200, 64, 2056, "bf16", api.MOE_TILE_AUTO, True),
    (1, 2, 2200, 1032, 1032, "bf16", api.MOE_TILE_SMALL, False),   # operands beyond an XCD's L2: runs in turn, a rest behind them
    (1, 2, 2200, 1032, 1032, "bf16", api.MOE_TILE_AUTO, True),
    (3, 2, 730, 1032, 1032, "bf16", api.MOE_TILE_AUTO, True),
    (1, 2, 700, 72, 520, "f32", api.MOE_TILE_AUTO, True),
    (1, 2, 1500, 712, 264, "f32", api.MOE_TILE_AUTO, False),       # 5 MB of operands in fp32
])
def test_tile_orders(n_src, G, C, M, H, dtype, tile, counted):
    """Every tile of a launch is computed once, in both orders in which the XCDs take them."""
    rng = np.random.default_rng(C + M)
    occ = rng.integers(C // 2, C + 1, size=(n_src, G)) if counted else None
    check_ffn(rng, n_src, G, C, M, H, dtype, tile, occ)


@pytest.mark.parametrize("n_src,C,rows", [
    (1, 512, None), (1, 513, None), (1, 512, (300, 514)), (1, 513, (300, 514)),           # one chunk
    (2, 256, (0, 257)), (2, 257, (0, 257)), (8, 64, None), (5, 103, None),                # a k tile of one chunk each
    (8, 64, (0, 65)), (5, 103, (0, 103)), (16, 32, (0, 33)), (41, 13, (0, 13)), (90, 21, (0, 22)),   # of pieces of several chunks
])
@pytest.mark.parametrize("tile", [api.MOE_TILE_256, api.MOE_TILE_192])
def test_weight_gradients_of_few_k_tiles(n_src, C, rows, tile):
    """256 x 256 weight-gradient tiles on both sides of the row count that decides their MFMA."""
    rng = np.random.default_rng(C + n_src)
    occ = rng.integers(rows[0], rows[1], size=(n_src, 2)) if rows else None
    check_ffn(rng, n_src, 2, C, 264, 520, "bf16", tile, occ)


@pytest.mark.parametrize("n_src,G,C,M,H,counted", [
    (1, 20, 1700, 72, 72, False),      # reductions in parts
    (1, 20, 1700, 72, 72, True),
    (6, 20, 300, 72, 136, True),       # packed chunks
    (1, 63, 600, 136, 72, True),       # whole reductions
])
def test_dx_beside_small_weight_gradients_and_alone(n_src, G, C, M, H, counted):
    """Weight gradients of 128 x 128 tiles whose dX has more than one round of tiles: a launch of its own."""
    rng = np.random.default_rng(C + G)
    occ = rng.integers(C // 2, C + 1, size=(n_src, G)) if counted else None
    check_ffn(rng, n_src, G, C, M, H, "bf16", api.MOE_TILE_AUTO, occ)
