"""se_prune_interval's compaction rounds: two are in flight, so the cases are
those where a round meets its neighbours: intervals around multiples of 64
slots, nothing kept, one slot kept or dropped, both work-group sizes (few units
and more than 256), both head sizes.  Moves are exact."""
import numpy as np
import pytest
import torch

from workloads import isolated_units, to_device

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("units,d", [(3, 128), (3, 64), (258, 64), (257, 128)])
@pytest.mark.parametrize("L,lo,hi,drop", [
    (64, 0, 64, "all"),            # the only round empties
    (65, 0, 64, "all"),            # one slot moves a whole round down
    (129, 63, 65, "all"),          # across the edge of two rounds
    (640, 1, 2, "all"),            # every later row moves by one
    (640, 64, 576, "odd"),         # whole rounds thinned to half
    (700, 100, 613, "first"),      # one slot of a long interval goes
    (700, 128, 640, "but one"),    # one stays
])
def test_mask_rounds(units, d, L, lo, hi, drop):
    import paper_2609_39068_amd as se
    host = isolated_units([L] * units, -(-L // 16), d, seed=L + hi, num_kv_heads=1)
    for u in range(units):          # slot s holds position s
        s = torch.arange(L)
        host.pos_pool[host.block_table[u, s // 16].long(), s % 16] = s.to(torch.int32)
    n = hi - lo
    i = torch.arange(n)
    stay = {"all": i < 0, "odd": i % 2 == 0, "first": i > 0, "but one": i == n // 2}[drop]
    keep = torch.cat([torch.arange(lo), lo + i[stay], torch.arange(hi, L)])
    gs = to_device(host, DEV)
    view = se.KVView(gs.kv_pool, gs.pos_pool, gs.score_pool, None, gs.block_table, gs.lengths, num_kv_heads=1)
    interval = torch.tensor([[lo, hi]] * units, dtype=torch.int32, device=DEV)
    mask = stay.to(torch.uint8).repeat(units, 1).to(DEV)
    count = torch.zeros(units, dtype=torch.int32, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    se.se_prune_interval(view, interval, mask, n, None, L, None, 0, count, err)
    torch.cuda.synchronize()
    assert se.se_read_device_errors(err) == 0
    Lp = len(keep)
    assert gs.lengths.tolist() == [Lp] * units
    assert count.tolist() == [-(-L // 16) - -(-Lp // 16)] * units
    to = torch.arange(Lp)
    for u in range(units):
        bt = host.block_table[u].long()
        for name in ("pos_pool", "score_pool"):
            a, b = getattr(gs, name).cpu()[bt[to // 16], to % 16], getattr(host, name)[bt[keep // 16], keep % 16]
            assert torch.equal(a, b), (name, u)
        if u < 2 or u == units - 1:
            kv = gs.kv_pool.cpu()
            for part in (0, 1):
                np.testing.assert_array_equal(kv[bt[to // 16], part, to % 16].view(torch.int16).numpy(),
                                              host.kv_pool[bt[keep // 16], part, keep % 16].view(torch.int16).numpy())
