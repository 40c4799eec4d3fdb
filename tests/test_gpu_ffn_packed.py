"""Expert FFN with row counts over many source chunks: k tiles of the weight gradients that are made of pieces of several
chunks, padding rows stored apart from the tiles (none, a few rows, most of the buffer), and reductions in parts."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2407_00599_amd import api, synth
from test_gpu_ffn import gpu_ffn
from test_gpu_ffn_gather import test_fused_dispatch_forward as fused_dispatch
from util import DEV, TOL, ROWS, EXPERT, to_dev, to_host, assert_close, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src,G,C,M,H,lo,hi,dtype", [
    (4, 2, 129, 264, 520, 0, 129, "bf16"),        # as few chunks as are packed
    (40, 1, 12, 136, 264, 0, 3, "bf16"),          # a k tile of twenty pieces and more, one tile in all
    (90, 2, 7, 72, 136, 0, 8, "bf16"),            # more than 64 chunks, a k tile across the sixty-fourth
    (5, 3, 64, 72, 136, 64, 65, "bf16"),          # no padding at all
    (6, 2, 700, 264, 520, 0, 2, "bf16"),          # almost nothing but padding
    (6, 20, 100, 64, 64, 0, 40, "bf16"),          # more than 16 experts
    (6, 2, 700, 72, 136, 0, 40, "f32"),
    (1, 2, 1700, 136, 264, 0, 1701, "bf16"),      # weight gradients in parts: a single chunk,
    (3, 1, 2100, 264, 520, 0, 2101, "bf16"),      # whole chunks,
    (30, 2, 300, 136, 264, 0, 301, "bf16"),       # packed chunks,
    (30, 2, 300, 72, 136, 0, 4, "bf16"),          # and more parts than k tiles
    (5, 16, 60, 264, 264, 0, 61, "bf16"),         # 256 x 256 weight gradients of the automatic plan (64 tiles)
    (12, 16, 60, 264, 264, 0, 61, "bf16"),
])
def test_packed_chunks(n_src, G, C, M, H, lo, hi, dtype):
    rng = np.random.default_rng(n_src * 1009 + C)
    occ = rng.integers(lo, hi, size=(n_src, G)).clip(0, C)
    Xn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    dYn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    pad = np.arange(C)[None, None, :] >= occ[:, :, None]
    Xn[pad] = 0; dYn[pad] = 0
    X, dY = synth.store(Xn, dtype), synth.store(dYn, dtype)
    W1 = synth.store((rng.standard_normal((G, M, H)) / np.sqrt(M)).astype(np.float32), dtype)
    W2 = synth.store((rng.standard_normal((G, H, M)) / np.sqrt(H)).astype(np.float32), dtype)
    cnt = torch.tensor(occ.astype(np.int32), device=DEV)
    got = gpu_ffn(*(to_dev(t) for t in (X, dY, W1, W2)), n_src, G, C, M, H, 0, 1, torch_dtype(dtype), cnt)
    rZ, rY = O.expert_ffn_fwd(X.val, W1.val, W2.val, 0, 1)
    rdX, rdW1, rdW2 = O.expert_ffn_bwd(dY.val, X.val, W1.val, W2.val, 0, 1)
    for name, t, ref, group in (("Z", got[0], rZ, ROWS), ("A", got[1], O.gelu(rZ), ROWS), ("Y", got[2], rY, ROWS),
                                ("dX", got[3], rdX, ROWS), ("dW1", got[4], rdW1, EXPERT), ("dW2", got[5], rdW2, EXPERT)):
        assert_close(to_host(t), ref, TOL[dtype], name, group)
    for t in got[:4]:
        assert np.all(to_host(t)[pad] == 0.0)
    again = gpu_ffn(*(to_dev(t) for t in (X, dY, W1, W2)), n_src, G, C, M, H, 0, 1, torch_dtype(dtype), cnt)
    for a, b in zip(got, again):
        assert torch.equal(a, b)      # the parts are added in order, nothing depends on when a workgroup runs


@pytest.mark.parametrize("fill", [0.05, 0.9])
def test_parts_through_a_slot_map(fill):
    """Weight gradients in parts whose rows come through a slot map: the bits of dispatch + FFN."""
    fused_dispatch(1800, 2, 2, 1700, 136, 264, 1, 0, "bf16", 0, fill, True)


@pytest.mark.parametrize("n_src,C,lo,hi", [(1, 1700, 900, 1701), (3, 1100, 0, 1101), (30, 120, 0, 121), (1, 1700, None, None)])
@pytest.mark.parametrize("esp_idx,whole", [(0, False), (1, False), (2, False), (1, True)])
def test_parts_of_a_hidden_shard(n_src, C, lo, hi, esp_idx, whole):
    """Reductions in parts that are added into columns / rows of the full gradient tensors; whole: with a workspace of dZ's
    size only, which the call accepts, the reductions are not cut."""
    G, M, H, n_esp = 2, 136, 408, 3
    Hl, hs = H // n_esp, slice(esp_idx * (H // n_esp), (esp_idx + 1) * (H // n_esp))
    rng = np.random.default_rng(n_src + esp_idx)
    occ = None if lo is None else rng.integers(lo, hi, size=(n_src, G))
    Xn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    dYn = rng.standard_normal((n_src, G, C, M)).astype(np.float32)
    if occ is not None:
        pad = np.arange(C)[None, None, :] >= occ[:, :, None]
        Xn[pad] = 0; dYn[pad] = 0
    X, dY = synth.store(Xn, "bf16"), synth.store(dYn, "bf16")
    W1 = synth.store((rng.standard_normal((G, M, H)) / np.sqrt(M)).astype(np.float32), "bf16")
    W2 = synth.store((rng.standard_normal((G, H, M)) / np.sqrt(H)).astype(np.float32), "bf16")
    full = api.moe_ffn_workspace_bytes(api.MOE_BF16, n_src, G, C, M, H, n_esp)
    dz = (n_src * G * C * Hl * 2 + 255) // 256 * 256
    assert full > dz          # the shape is one whose reductions are cut
    cnt = None if occ is None else torch.tensor(occ.astype(np.int32), device=DEV)
    got = gpu_ffn(*(to_dev(t) for t in (X, dY, W1, W2)), n_src, G, C, M, H, esp_idx, n_esp, torch.bfloat16, cnt,
                  ws_bytes=dz if whole else full)
    rdX, rdW1, rdW2 = O.expert_ffn_bwd(dY.val, X.val, W1.val, W2.val, esp_idx, n_esp)
    hW1, hW2 = to_host(got[4]), to_host(got[5])
    assert_close(to_host(got[3]), rdX, TOL["bf16"], "dX", ROWS)
    assert_close(hW1[:, :, hs], rdW1, TOL["bf16"], "dW1", EXPERT)
    assert_close(hW2[:, hs, :], rdW2, TOL["bf16"], "dW2", EXPERT)
    others = np.ones(H, bool)
    others[hs] = False
    assert np.all(hW1[:, :, others] == 3.0) and np.all(hW2[:, others, :] == 3.0)
