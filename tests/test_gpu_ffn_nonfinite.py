"""GPU: infinities in the expert FFN's operands.  A k tile that is only partly inside the problem must add nothing for the
rows it lacks: zero times whatever stands in for them in the other operand would turn an infinite sum into NaN.  All
finite operands are positive, so an output whose sum holds the infinity is +inf, and every other output must have the bits
of the run without it."""
import pytest
import torch

from paper_2407_00599_amd import api
from util import DEV, torch_dtype

pytestmark = pytest.mark.gpu

INF = float("inf")
N_SRC, G, C, M, H = 2, 2, 70, 72, 200      # 70 rows, 72 and 200 columns: k tiles of 64 with 6 and 8 values left
ROW, MCOL, HCOL = 64, 64, 192              # the first of those


def expect(got, finite, inf_at, name):
    want = finite.clone()
    want[inf_at] = INF
    assert torch.equal(got, want), (name, int(got.isnan().sum()), int((got != want).sum()))


NOTHING = (slice(0, 0),)


@pytest.mark.parametrize("dtype,tile", [("bf16", api.MOE_TILE_AUTO), ("bf16", api.MOE_TILE_SMALL), ("bf16", api.MOE_TILE_256),
                                        ("bf16", api.MOE_TILE_192), ("f32", api.MOE_TILE_AUTO)])
@pytest.mark.parametrize("n_src,gather", [(N_SRC, False), (1, False), (1, True)])
def test_infinity_in_the_first_row_of_a_partial_k_tile(n_src, gather, dtype, tile):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    tdt = torch_dtype(dtype)
    positive = lambda *s: (torch.rand(*s, generator=gen, device=DEV) + 0.1).to(tdt)      # noqa: E731
    X, dY = positive(n_src, G, C, M), positive(n_src, G, C, M)
    W1, W2 = positive(G, M, H) / M, positive(G, H, M) / H
    inv = torch.arange(G * C, dtype=torch.int32, device=DEV).reshape(G, C)
    dt = api.MOE_BF16 if dtype == "bf16" else api.MOE_F32
    ws = torch.empty(api.moe_ffn_workspace_bytes(dt, n_src, G, C, M, H, 1), dtype=torch.uint8, device=DEV)

    def fwd(w1, w2):
        Z, A, Y = (torch.empty(n_src, G, C, n, dtype=tdt, device=DEV) for n in (H, H, M))
        if gather:
            api.moe_expert_ffn_fwd_gather(X.view(G * C, M), inv, G * C, 1, w1, w2, G, C, M, H, 0, 1, Z, A, Y, None, tile)
        else:
            api.moe_expert_ffn_fwd(X, w1, w2, n_src, G, C, M, H, 0, 1, Z, A, Y, None, tile)
        return Z, A, Y

    def bwd(Z, A, dy, w1, w2):
        dX, dW1, dW2 = torch.empty_like(X), torch.empty_like(W1), torch.empty_like(W2)
        if gather:
            api.moe_expert_ffn_bwd_gather(dy, X.view(G * C, M), inv, G * C, 1, Z, A, w1, w2, G, C, M, H, 0, 1, dX, dW1, dW2, ws,
                                          None, tile)
        else:
            api.moe_expert_ffn_bwd(dy, X, Z, A, w1, w2, n_src, G, C, M, H, 0, 1, dX, dW1, dW2, ws, None, tile)
        return dX, dW1, dW2

    def with_inf(t, *at):
        t = t.clone()
        t[at] = INF
        return t

    a = slice(None)
    Z, A, Y = fwd(W1, W2)
    dX, dW1, dW2 = bwd(Z, A, dY, W1, W2)
    for t in (Z, A, Y, dX, dW1, dW2):
        assert t.isfinite().all() and (t > 0).all()

    z, act, y = fwd(with_inf(W1, 1, MCOL, 5), W2)                 # Z = X W1
    expect(z, Z, (a, 1, a, 5), "Z"), expect(act, A, (a, 1, a, 5), "A"), expect(y, Y, (a, 1), "Y")
    z, act, y = fwd(W1, with_inf(W2, 1, HCOL, 7))                 # Y = A W2
    expect(z, Z, NOTHING, "Z"), expect(act, A, NOTHING, "A"), expect(y, Y, (a, 1, a, 7), "Y")

    s = n_src - 1
    dx, dw1, dw2 = bwd(Z, A, with_inf(dY, s, 0, ROW, 3), W1, W2)  # dW2 = A^T dY, dW1 = X^T dZ: a chunk's last rows
    expect(dx, dX, (s, 0, ROW), "dX"), expect(dw1, dW1, (0,), "dW1"), expect(dw2, dW2, (0, a, 3), "dW2")
    dx, dw1, dw2 = bwd(Z, A, dY, W1, with_inf(W2, 1, 5, MCOL))    # dA = dY W2^T
    expect(dx, dX, (a, 1), "dX"), expect(dw1, dW1, (1, a, 5), "dW1"), expect(dw2, dW2, NOTHING, "dW2")
    dx, dw1, dw2 = bwd(Z, A, dY, with_inf(W1, 1, 9, HCOL), W2)    # dX = dZ W1^T
    expect(dx, dX, (a, 1, a, 9), "dX"), expect(dw1, dW1, NOTHING, "dW1"), expect(dw2, dW2, NOTHING, "dW2")
