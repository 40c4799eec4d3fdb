"""GPU parity: gate logits at the edges of the kernels' tiles and of the rules that choose between them."""
import numpy as np
import pytest
import torch

from paper_2407_00599_amd import api
from util import DEV

pytestmark = pytest.mark.gpu


def gate(x, Wg, bias):
    S, M = x.shape
    E, k, C = Wg.shape[1], 1, S
    i32 = torch.int32
    logits = torch.full((S, E), float("nan"), device=DEV)
    idx, slot, inv = (torch.empty(n, dtype=i32, device=DEV) for n in ((S, k), (S, k), (E, C)))
    w, counts = torch.empty(S, k, device=DEV), torch.empty(E, dtype=i32, device=DEV)
    ws = torch.empty(api.moe_gate_workspace_bytes(S, E, k), dtype=torch.uint8, device=DEV)
    api.moe_gate_topk(x, Wg, bias, S, M, E, k, C, 0, 1, 0, logits, idx, slot, w, inv, counts, ws)
    torch.cuda.synchronize()
    return logits


# up to 16 experts: walks of a few waves (few tokens for their M), 16 x 16 tiles, the 4-block form (many bf16 tokens); beyond:
# 16 x 16 tiles up to 128 tiles of 64 x 64, four groups over M up to 256, two beyond; M around whole chunks of 32 (tails of 8,
# 16, 24), fewer chunks than waves or groups
@pytest.mark.parametrize("S,M,E", [
    (1, 8, 1), (1023, 1024, 8), (1024, 1024, 8), (2049, 264, 3), (511, 520, 12), (513, 520, 12), (1003, 520, 16), (8191, 2048, 16),
    (8192, 136, 4), (8193, 40, 5), (16383, 72, 8), (16384, 72, 8), (16390, 1032, 9), (40000, 24, 16),
    (15, 64, 17), (17, 200, 33), (64, 2056, 256), (300, 8, 65), (8192, 96, 64), (8193, 40, 64), (8200, 264, 17), (16384, 24, 64),
    (4160, 104, 256), (17000, 8, 20), (16400, 232, 130),
])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_logits(S, M, E, dtype):
    g = torch.Generator(device=DEV)
    g.manual_seed(S + M + E)
    x = torch.randn(S, M, generator=g, device=DEV).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    Wg, bias = torch.randn(M, E, generator=g, device=DEV), torch.randn(E, generator=g, device=DEV)
    exact = x.double() @ Wg.double() + bias.double()
    got = gate(x, Wg, bias)
    # fp64 sums of M products, rounded once: M 2^-53 sum |x w| and half a place of the result
    bound = exact.abs() * 2.0 ** -24 + (M + 2) * 2.0 ** -53 * (x.double().abs() @ Wg.double().abs() + bias.abs().double())
    assert bool(((got.double() - exact).abs() <= bound).all())


@pytest.mark.parametrize("S,M,E", [(300, 40, 20), (8200, 40, 64), (16500, 136, 64), (1100, 72, 12), (16384, 72, 8)])
def test_non_finite_values_stay_in_their_row_and_column(S, M, E):
    """Tokens, experts and values of k past the end are fetched from other places; what lies there must not matter."""
    g = torch.Generator(device=DEV)
    g.manual_seed(S)
    x, Wg = torch.randn(S, M, generator=g, device=DEV).to(torch.bfloat16), torch.randn(M, E, generator=g, device=DEV)
    want = gate(x, Wg, None)
    x[S - 1], x[S // 2, 0], x[7, M - 1] = float("inf"), float("nan"), float("-inf")
    Wg[:, E - 1] = float("nan")
    got = gate(x, Wg, None)
    rows = torch.ones(S, dtype=torch.bool, device=DEV)
    rows[[S - 1, S // 2, 7]] = False
    assert torch.equal(got[rows][:, :E - 1], want[rows][:, :E - 1])
    assert not bool(torch.isfinite(got[~rows]).any()) and not bool(torch.isfinite(got[:, E - 1]).any())
