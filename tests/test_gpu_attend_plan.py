"""The query-tile plan of the prefill attention on both sides of its rule (a
scan of the list, a binary search above 4096 entries): sequences that left the
list, one entry, lists that end on a tile, more sequences than a wave has
lanes.  Causal attention against plain torch in 64 bits."""
import math

import numpy as np
import pytest
import torch

from paper_2601_03700_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n_seq,length,keep,gone", [(1, 5, 1.0, ()), (3, 128, 1.0, ()),
                                                    (5, 200, 0.6, (0, 2)), (70, 14, 0.9, (3, 69)),
                                                    (4, 1024, 1.0, ()), (5, 1024, 0.79, (4,)),
                                                    (4, 1040, 1.0, (1,)), (9, 520, 0.95, (0, 8))])
def test_tiles(n_seq, length, keep, gone):
    _tiles(n_seq, length, keep, gone, False)


# more than 4096 entries: the first or the last sequence gone, one entry past the
# line, sequences that end on a tile, more sequences than a wave has lanes
@pytest.mark.parametrize("n_seq,length,keep,gone", [(1, 4097, 1.0, ()), (5, 1025, 1.0, (0,)),
                                                    (9, 640, 1.0, (0, 8)), (6, 1024, 0.9, (5,)),
                                                    (130, 40, 0.95, (0, 64, 129))])
def test_tiles_of_long_lists(n_seq, length, keep, gone):
    _tiles(n_seq, length, keep, gone, True)


def _tiles(n_seq, length, keep, gone, searched):
    print(f"attention plan {n_seq}x{length} keep={keep} gone={gone}", flush=True)
    H, hd = 2, 64
    rng = np.random.default_rng(n_seq * length)
    n_tok = n_seq * length
    live = rng.random(n_tok) < keep
    live[length - 1] = True
    for b in gone:
        live[b * length:(b + 1) * length] = False
    live[n_tok // 2] = True
    act = np.flatnonzero(live).astype(np.int32)
    n = act.size
    assert (n > 4096) == searched   # the plan's line between scan and search
    i32 = dict(dtype=torch.int32, device=DEV)
    pos = torch.arange(length, **i32).repeat(n_seq)
    seq = torch.arange(n_seq, **i32).repeat_interleave(length)
    g = torch.Generator(device=DEV).manual_seed(n)
    q, k, v = (torch.randn((m, H, hd), generator=g, device=DEV).to(torch.bfloat16)
               for m in (n_tok, n_tok, n_tok))
    rows = torch.full((n_tok,), -5, **i32)         # past the count: never read
    rows[:n] = torch.from_numpy(act).to(DEV)
    cnt = torch.tensor([n], **i32)
    out = torch.full((n_tok, H, hd), 7.0, dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(B.attend_workspace_bytes(n_tok, n_seq, H, hd, length), dtype=torch.uint8, device=DEV)
    B.attend(H, hd, q, rows, cnt, n_tok, pos, seq, n_seq, k, v, length, out, causal=True, workspace=ws)
    assert (out[n:] == 7.0).all()
    at = torch.from_numpy(act).to(DEV).long()
    for b in range(n_seq):
        mine = torch.nonzero(seq[at] == b).flatten()
        if mine.numel() == 0:
            continue
        p = pos[at[mine]].long()
        s = slice(b * length, (b + 1) * length)
        sc = torch.einsum("thd,shd->hts", q[mine].double().cpu(), k[s].double().cpu()) / math.sqrt(hd)
        mask = torch.arange(length)[None, :] <= p.cpu()[:, None]
        w = torch.softmax(sc.masked_fill(~mask, -math.inf), -1)
        ref = torch.einsum("hts,shd->thd", w, v[s].double().cpu())
        # bf16 keeps 8 bits: each weight is off by up to 2^-8 of itself, in the sum and
        # in the normaliser, and so is the result: |err| <= 2^-8 (sum w |v| + 2 |o|);
        # f32 scores and sums add about 1e-5
        wv = torch.einsum("hts,shd->thd", w, v[s].double().cpu().abs())
        err = (out[mine].double().cpu() - ref).abs()
        assert (err / (2.0 ** -8 * (wv + 2 * ref.abs()) + 1e-4)).max() <= 1.0
