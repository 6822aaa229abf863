"""se_omnikv_select where the selection starts from a sampled threshold: the
edges of its range, score distributions that the sample judges well, badly and
not at all, and ties at the threshold.  The selection is a selection of given
numbers, so it is exact against a stable sort."""
import numpy as np
import pytest
import torch

from workloads import isolated_units, to_device

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _scores(kind, n, g):
    if kind == "normal":
        return torch.randn(n, generator=g)
    if kind == "levels":        # a thousand values: ties at the threshold
        return torch.randint(0, 1000, (n,), generator=g).float() / 7
    if kind == "recent":        # every large score in the last slots
        return torch.arange(n).float() ** 2 / n + torch.rand(n, generator=g)
    if kind == "period":        # the sampled slots (equal distances) are the lowest: far too many pass
        s = torch.rand(n, generator=g) + 1.0
        s[(torch.arange(1024) * n) // 1024] = -1.0
        return s
    if kind == "few":           # the sampled slots are the largest: too few pass
        s = torch.rand(n, generator=g)
        s[(torch.arange(1024) * n) // 1024] += 10.0
        return s
    if kind == "equal":
        return torch.full((n,), 2.5)
    s = torch.randn(n, generator=g)     # "edges": infinities, both zeros, the smallest numbers
    s[::5] = -float("inf")
    s[1::97] = float("inf")
    s[2::7] = -0.0
    s[3::7] = 0.0
    s[4::11] = 1e-42
    return s


@pytest.mark.parametrize("kind", ["normal", "levels", "recent", "period", "few", "equal", "edges"])
@pytest.mark.parametrize("L,budget", [
    (4095, 100),        # just below the range
    (4096, 1365),       # the shortest, and nearly a third of it
    (4099, 1),
    (36869, 8192),
    (131072, 2048),     # the longest
    (131073, 2048),     # past it
])
def test_selection_matches_a_stable_sort(L, budget, kind):
    import paper_2609_39068_amd as se
    hkv, G, nreq = 2, 1, 2
    stride = (L + 3) // 4 * 4
    g = torch.Generator().manual_seed(L + budget)
    logits = torch.full((nreq * hkv, stride), 99.0)
    want = []
    for r in range(nreq):
        s = _scores(kind, L, g)
        logits[r * hkv, :L] = s                                   # one head holds the score, the other is below it
        logits[r * hkv + 1, :L] = torch.where(torch.isinf(s), s, s - s.abs() - 1.0)
        best = torch.maximum(logits[r * hkv, :L], logits[r * hkv + 1, :L]).numpy() + 0.0
        want.append(np.sort(np.argsort(-best, kind="stable")[:budget]))
    st = to_device(isolated_units([L] * (nreq * hkv), (L + 15) // 16, 64, 1, num_kv_heads=hkv, with_scores=False), DEV)
    view = se.KVView(st.kv_pool, st.pos_pool, None, None, st.block_table, st.lengths, num_kv_heads=hkv)
    sel = torch.empty((nreq, budget), dtype=torch.int32, device=DEV)
    ws = torch.empty(se.se_workspace_bytes(se.SE_OP_OMNIKV_SELECT, nreq, L, (L + 15) // 16, G, 64, 0), dtype=torch.uint8, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    se.se_omnikv_select(view, G, logits.to(DEV), stride, budget, L, sel, ws, err)
    torch.cuda.synchronize()
    assert se.se_read_device_errors(err) == 0
    for r in range(nreq):
        np.testing.assert_array_equal(sel[r].cpu().numpy(), want[r])
