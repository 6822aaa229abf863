"""The logits output of se_decode_attend and the per-group maximum of the OmniKV
observation layer: stored in bursts of pages, which a wavefront takes singly
or in groups of four by the length of the unit.  Logits against float64; the
maximum against the logits, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2609_39068_amd import _binding
from workloads import isolated_units, to_device

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("stride_pad", [0, 3])    # 16-byte aligned rows, and not
@pytest.mark.parametrize("G,d,lengths", [
    (4, 128, [15, 1, 300, 16 * 127 + 9]),         # one page up to just below groups of four
    (4, 128, [16 * 128, 16 * 129 + 1, 5003, 16 * 131]),   # just above, ends inside a group
    (8, 64, [4000, 2500]),
    (2, 128, [3333, 17]),
    (1, 64, [9000, 9001]),                        # split over work-groups
    (4, 64, [2000] * 300),                        # more than one work-group per compute unit: 512 threads
])
def test_logits_and_group_maximum(G, d, lengths, stride_pad):
    import paper_2609_39068_amd as se
    U = len(lengths)
    P = -(-max(lengths) // 16)
    host = isolated_units(lengths, P, d, seed=G + d + U, num_kv_heads=1, with_scores=False)
    gs = to_device(host, DEV)
    view = se.KVView(gs.kv_pool, gs.pos_pool, None, None, gs.block_table, gs.lengths, num_kv_heads=1)
    q = torch.randn((U, G, d), generator=torch.Generator().manual_seed(2)).to(torch.bfloat16)
    ml = max(lengths)
    stride = -(-ml // 64) * 64 + stride_pad
    scale = float(np.float32(1 / np.sqrt(d)))
    ws = torch.empty(max(1, se.se_workspace_bytes(se.SE_OP_DECODE_ATTEND, U, ml, P, G, d, 0)), dtype=torch.uint8, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    out, out2 = torch.zeros(U, G, d, device=DEV), torch.zeros(U, G, d, device=DEV)
    logits = torch.full((U, G, stride), 77.0, device=DEV)
    gmax = torch.full((U, stride), 77.0, device=DEV)
    se.se_decode_attend(view, G, q.to(DEV), None, None, None, None, 0, scale, ml, 0, out, None, logits, stride, ws, err)
    _binding._observe_attend(view, G, q.to(DEV), None, None, None, scale, ml, out2, None, gmax, stride, ws, err)
    torch.cuda.synchronize()
    assert se.se_read_device_errors(err) == 0
    assert torch.equal(out, out2)
    lg, gm = logits.cpu(), gmax.cpu()
    for u in range(0, U, max(1, U // 8)):
        L = lengths[u]
        k = host.kv_pool[host.block_table[u, :-(-L // 16)].long(), 0].reshape(-1, d)[:L].double()
        want = scale * (q[u].double() @ k.T)
        # d exact products summed in fp32: a few 2^-24 of the sum of magnitudes
        assert torch.allclose(lg[u, :, :L].double(), want, rtol=1e-5, atol=1e-5), u
        assert torch.equal(gm[u, :L], lg[u, :, :L].amax(0)), u
        assert bool((lg[u, :, L:] == 77.0).all()) and bool((gm[u, L:] == 77.0).all()), u   # nothing past the length
