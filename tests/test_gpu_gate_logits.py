"""GPU parity: gate logits at the edges of the kernels' tiles and of the rules that choose between them."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2407_00599_amd import api
from util import DEV, rel_err, to_host

pytestmark = pytest.mark.gpu


def gate(x, Wg, bias, k=1, C=None, norm=0, everything=False):
    S, M = x.shape
    E, C = Wg.shape[1], C or S
    i32 = torch.int32
    logits = torch.full((S, E), float("nan"), device=DEV)
    idx, slot, inv = (torch.empty(n, dtype=i32, device=DEV) for n in ((S, k), (S, k), (E, C)))
    w, counts = torch.empty(S, k, device=DEV), torch.empty(E, dtype=i32, device=DEV)
    ws = torch.empty(api.moe_gate_workspace_bytes(S, E, k), dtype=torch.uint8, device=DEV)
    api.moe_gate_topk(x, Wg, bias, S, M, E, k, C, 0, 1, norm, logits, idx, slot, w, inv, counts, ws)
    torch.cuda.synchronize()
    return (logits, idx, slot, inv, w, counts) if everything else logits


# up to 16 experts: walks of a few waves (few tokens for their M), 16 x 16 tiles, the 4-block form (many bf16 tokens); beyond:
# 16 x 16 tiles up to 128 tiles of 64 x 64, one, two or four groups over M beyond; M around whole chunks of 32 (tails of 8,
# 16, 24), fewer chunks than waves or groups
@pytest.mark.parametrize("S,M,E", [
    (1, 8, 1), (1023, 1024, 8), (1024, 1024, 8), (2049, 264, 3), (511, 520, 12), (513, 520, 12), (1003, 520, 16), (8191, 2048, 16),
    (1, 1440, 16), (1, 1448, 16), (512, 1176, 13), (513, 2048, 16), (1023, 4096, 12), (1000, 3072, 9), (1000, 3072, 10), (1640, 3072, 14), (1641, 3080, 14),
    (2048, 3072, 9), (2049, 3072, 9),
    (2048, 2048, 8), (2049, 2048, 8), (3400, 2056, 5), (3401, 2056, 5), (4096, 2048, 2), (4097, 1536, 7), (5400, 1544, 3), (5401, 1544, 3), (7000, 1536, 4), (7001, 1536, 4), (8191, 3072, 1),
    (8192, 512, 8), (8193, 512, 8), (8193, 504, 8), (8200, 1032, 5),
    (8192, 136, 4), (8193, 40, 5), (16383, 72, 8), (16384, 72, 8), (16390, 1032, 9), (40000, 24, 16),
    (15, 64, 17), (17, 200, 33), (64, 2056, 256), (300, 8, 65), (8192, 96, 64), (8193, 40, 64), (8200, 264, 17), (16384, 24, 64),
    (4160, 104, 256), (17000, 8, 20), (16400, 232, 130),
    # short M: 1024 blocks of 16 x 16 and more; one group up to 248, two from 256, four from 384 up to 256 blocks of 64 x 64
    (8192, 64, 32), (8193, 64, 32), (8192, 64, 48), (8200, 16, 17), (8200, 72, 24), (8200, 248, 40), (8200, 256, 40), (8200, 376, 17),
    (8200, 384, 17), (9000, 248, 128), (9000, 256, 128),
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


# the experts selected by the logits kernel (up to 16 experts, k <= 3, S k <= 6144 or 8192), and one step beyond each line; ties by equal columns
@pytest.mark.parametrize("S,M,E,k,C,norm", [
    (1, 8, 1, 1, 1, 0), (63, 64, 16, 3, 5, 1), (65, 2048, 8, 2, 9, 0), (257, 40, 3, 3, 200, 1), (1023, 520, 12, 3, 250, 1),
    (2049, 72, 16, 2, 300, 0), (2730, 64, 9, 3, 1000, 1), (2731, 64, 9, 3, 900, 0), (4096, 1024, 8, 2, 1100, 1), (4097, 64, 8, 2, 1000, 1),
    (8191, 24, 2, 1, 4000, 0), (8192, 136, 12, 1, 600, 0), (300, 64, 16, 4, 70, 1),
    (6144, 24, 5, 1, 900, 0), (6145, 24, 5, 1, 900, 0), (2048, 64, 9, 3, 700, 1), (2049, 64, 9, 3, 700, 1), (4096, 24, 9, 2, 900, 1),
    # as many tokens as gate_topk's one block is left with, and one more
    (256, 64, 4, 1, 70, 0), (257, 64, 4, 2, 100, 1), (64, 64, 8, 1, 9, 0), (65, 64, 5, 3, 20, 0), (112, 72, 9, 3, 30, 1), (113, 72, 9, 3, 30, 1),
])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_routing(S, M, E, k, C, norm, dtype):
    g = torch.Generator(device=DEV)
    g.manual_seed(S + E)
    x = torch.randn(S, M, generator=g, device=DEV).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    Wg = torch.randn(M, E, generator=g, device=DEV) * 0.1
    if E > 4:
        Wg[:, 4] = Wg[:, 1]
    logits, idx, slot, inv, w, counts = (to_host(t) for t in gate(x, Wg, torch.linspace(1, 0, E, device=DEV).index_fill(0, torch.tensor(
        [min(4, E - 1)], device=DEV), 1 - 1 / max(E - 1, 1)) if E > 4 else None, k, C, norm, True))
    logits = logits.astype(np.float32)
    want = O.topk_select(logits, k)
    assert np.array_equal(idx, want)
    for got, ref in zip((slot, inv, counts), O.capacity_slots(want, E, C)):
        assert np.array_equal(got, ref)
    assert rel_err(w, O.combine_weights(logits, want, bool(norm))) <= 1e-5
