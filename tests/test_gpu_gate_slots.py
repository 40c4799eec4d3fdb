"""GPU: the slots of the gate where every block adds up the histograms itself, up to the largest of these and just beyond, against the
choice-major queues that the returned choices make."""
import pytest
import torch

from paper_2407_00599_amd import api
from util import DEV

pytestmark = pytest.mark.gpu


# (choice, expert) pairs in fours and not, rows of one, four, sixteen and more per thread, more units than threads, demand of more than
# 16 bits hold over all blocks; the last block partly filled; 256 KiB of histograms and 64 MiB over all blocks, and one block more
@pytest.mark.parametrize("S,E,k,hot", [
    (2000, 17, 3, False), (65 * 64, 64, 8, False), (8192 + 1, 128, 4, True), (128 * 64, 256, 8, False), (128 * 64 + 1, 256, 8, False),
    (70000, 16, 2, True), (73280, 51, 1, True), (1024 * 64, 16, 4, False), (1024 * 64 + 3, 16, 4, True), (300, 255, 7, False), (12000, 2, 1, True),
    (30000, 257 // 3, 3, False), (131072, 4, 1, True),
    # a wave's sums added across its lanes: one, four and eight pairs; more than 65535 of a pair to a wave; two and twelve pairs are not
    (9000, 1, 1, False), (524288 - 5, 1, 1, False), (20000, 4, 1, False), (9001, 2, 2, False), (30000, 8, 1, True), (131072, 2, 1, True), (9000, 4, 3, False),
])
def test_slots(S, E, k, hot):
    g = torch.Generator(device=DEV)
    g.manual_seed(S + E)
    x = torch.randn(S, 8, generator=g, device=DEV)
    Wg = torch.randn(8, E, generator=g, device=DEV) * 0.5
    bias = torch.zeros(E, device=DEV)
    if hot:
        bias[E // 2] = 50.0
    C = max(1, S * k // E * 5 // 4)
    i32 = dict(dtype=torch.int32, device=DEV)
    logits, w = torch.empty(S, E, device=DEV), torch.empty(S, k, device=DEV)
    idx, slot = torch.full((S, k), -7, **i32), torch.full((S, k), -7, **i32)
    inv, counts = torch.full((E, C), -7, **i32), torch.full((E,), -7, **i32)
    ws = torch.full((api.moe_gate_workspace_bytes(S, E, k),), 255, dtype=torch.uint8, device=DEV)
    api.moe_gate_topk(x, Wg, bias, S, 8, E, k, C, 0, 1, 1, logits, idx, slot, w, inv, counts, ws)
    torch.cuda.synchronize()
    queue = idx.long().T.reshape(-1)                       # choice-major
    order = torch.sort(queue, stable=True)[1]
    total = torch.bincount(queue, minlength=E)
    first = torch.cumsum(total, 0) - total
    pos = torch.empty_like(queue)
    pos[order] = torch.arange(S * k, device=DEV) - first[queue[order]]
    want = torch.where(pos < C, pos, -1).view(k, S).T
    assert torch.equal(counts.long(), total) and torch.equal(slot.long(), want)
    t, j = torch.nonzero(want >= 0, as_tuple=True)
    winv = torch.full((E, C), -1, dtype=torch.int64, device=DEV)
    winv[idx.long()[t, j], want[t, j]] = t * k + j
    assert torch.equal(inv.long(), winv)
