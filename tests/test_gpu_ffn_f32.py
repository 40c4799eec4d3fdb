"""GPU parity of the fp32 expert FFN at the edges of its tiles (32 and 64 rows and columns, k chunks of 32 in pairs): every product
against the float64 product of the operands that the call was given or returned."""
import pytest
import torch

from paper_2407_00599_amd import api
from util import DEV

pytestmark = pytest.mark.gpu


def close(got, A, B, name):
    """got = A B, summed in float64 and rounded once: K 2^-53 of the sum of magnitudes and half a place of the result."""
    A, B = A.double(), B.double()
    exact, size = A @ B, A.abs() @ B.abs()
    assert bool(((got.double() - exact).abs() <= exact.abs() * 2.0 ** -24 + (A.shape[-1] + 2) * 2.0 ** -53 * size).all()), name


def run(n_src, G, C, M, H, occ, gather):
    g = torch.Generator(device=DEV)
    g.manual_seed(C + M + H)
    rn = lambda *s: torch.randn(*s, generator=g, device=DEV)      # noqa: E731
    W1, W2, dY = rn(G, M, H) / M ** 0.5, rn(G, H, M) / H ** 0.5, rn(n_src, G, C, M)
    counts = None if occ is None else torch.tensor(occ, dtype=torch.int32, device=DEV).expand(n_src, G).contiguous()
    pad = torch.zeros(n_src, G, C, dtype=torch.bool, device=DEV)
    if counts is not None:
        pad = torch.arange(C, device=DEV) >= counts[:, :, None]
    nan = lambda *s: torch.full(s, float("nan"), device=DEV)      # noqa: E731
    Z, A, Y, dX, dW1, dW2 = nan(n_src, G, C, H), nan(n_src, G, C, H), nan(n_src, G, C, M), nan(n_src, G, C, M), nan(G, M, H), nan(G, H, M)
    nbytes = api.moe_ffn_workspace_bytes(api.MOE_F32, n_src, G, C, M, H, 1)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=DEV)
    if gather:
        S, k = G * C, 2
        x = rn(S, M)
        inv = torch.randint(0, S * k, (G, C), generator=g, device=DEV, dtype=torch.int32)
        inv[pad[0]] = -1
        inv[:, ::7] = -1
        X = torch.where(inv[..., None] >= 0, x[inv.clamp(min=0) // k], 0)[None]
        dY[(inv < 0)[None]] = 0
        api.moe_expert_ffn_fwd_gather(x, inv, S, k, W1, W2, G, C, M, H, 0, 1, Z, A, Y, counts)
        api.moe_expert_ffn_bwd_gather(dY, x, inv, S, k, Z, A, W1, W2, G, C, M, H, 0, 1, dX, dW1, dW2, ws, counts)
    else:
        X = rn(n_src, G, C, M)
        X[pad] = 0
        dY[pad] = 0
        api.moe_expert_ffn_fwd(X, W1, W2, n_src, G, C, M, H, 0, 1, Z, A, Y, counts)
        api.moe_expert_ffn_bwd(dY, X, Z, A, W1, W2, n_src, G, C, M, H, 0, 1, dX, dW1, dW2, ws, counts)
    torch.cuda.synchronize()
    dZ = ws[:n_src * G * C * H * 4].view(torch.float32).view(n_src, G, C, H).clone()
    dZ[pad] = 0                                                    # (not written, not read)
    for t in (Z, A, Y, dX):
        assert not bool(t[pad].any())
    rows = lambda t, e: t[:, e].reshape(n_src * C, -1)             # noqa: E731
    for e in range(G):
        close(rows(Z, e), rows(X, e), W1[e], "Z"), close(rows(Y, e), rows(A, e), W2[e], "Y")
        close(dW2[e], rows(A, e).T, rows(dY, e), "dW2"), close(dW1[e], rows(X, e).T, rows(dZ, e), "dW1")
        close(rows(dX, e), rows(dZ, e), W1[e].T, "dX")


@pytest.mark.parametrize("n_src,G,C,M,H,occ", [
    (1, 1, 1, 8, 8, None), (1, 2, 31, 24, 40, None), (1, 2, 33, 32, 72, [33, 20]), (1, 3, 65, 40, 96, [0, 64, 65]),
    (3, 2, 50, 104, 64, [17, 50]), (1, 2, 97, 96, 136, [97, 33]), (70, 1, 9, 64, 40, [5]),
    # enough tiles for 64 x 64: whole and ragged rows and columns, odd and even numbers of chunks
    (1, 8, 64, 72, 6208, None), (1, 5, 300, 2056, 2088, [300, 257, 64, 0, 130]), (2, 4, 400, 1024, 264, [400, 1, 333, 64]),
    # 64 x 64: one, two and three chunks of k; weight gradients over none to four
    (1, 8, 128, 32, 3200, [128, 0, 20, 33, 64, 65, 96, 97]), (1, 8, 128, 64, 3168, None), (1, 8, 128, 96, 3104, [128] * 7 + [1]),
])
@pytest.mark.parametrize("gather", [False, True])
def test_products(n_src, G, C, M, H, occ, gather):
    if gather and n_src > 1:
        pytest.skip("one chunk per expert")
    run(n_src, G, C, M, H, occ, gather)


def test_leading_dimension_beyond_32_bit_offsets():
    run(1, 1, 3, 1 << 24, 8, [2], False)
