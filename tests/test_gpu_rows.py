"""Row kernels with a 16-byte form and an element form: both sides of the rule
(row length, alignment), against plain torch."""
import pytest
import torch

from paper_2601_03700_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rows(n, d, dtype, off=0, seed=0):
    """[n, d] whose data starts `off` elements after a 16-byte boundary."""
    g = torch.Generator(device=DEV).manual_seed(seed + d)
    flat = torch.randn(n * d + off, generator=g, device=DEV).to(dtype)
    return flat[off:].view(n, d)


def _ids(n, hi):
    ids = (torch.arange(n, device=DEV) * 37 % hi).to(torch.int32)
    ids[0], ids[-1] = -3, hi + 5        # clamped into the table
    return ids, ids.clamp(0, hi - 1).long()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,off", [(4, 0), (8, 0), (12, 0), (100, 0), (768, 0), (768, 1), (4096, 0)])
def test_embed(dtype, d, off):
    ids, at = _ids(67, 29)
    table = _rows(29, d, dtype, off)
    out = torch.full((67, d), -7.0, dtype=dtype, device=DEV)
    B.embed(67, d, 29, ids, table, out)
    assert torch.equal(out, table[at])
    wpe = _rows(11, d, dtype, off, seed=1)
    pos, pat = _ids(67, 11)
    B.embed_positions(67, d, 29, 11, ids, pos, table, wpe, out)
    assert torch.equal(out, (table[at].float() + wpe[pat].float()).to(dtype))


@pytest.mark.parametrize("d,off", [(8, 0), (100, 0), (512, 0), (768, 0), (768, 4), (1024, 0), (2056, 0)])
def test_encoder_embed(d, off):
    bf = torch.bfloat16
    ids, at = _ids(45, 31)
    pos, pat = _ids(45, 9)
    word, pemb = _rows(31, d, bf, off), _rows(9, d, bf, off, seed=1)
    temb, g, b = (_rows(1, d, bf, off, seed=s)[0] for s in (2, 3, 4))
    out = torch.empty((45, d), dtype=bf, device=DEV)
    B.encoder_embed(45, d, 31, 9, 1e-12, ids, pos, word, pemb, temb, g, b, out)
    x = word[at].double() + pemb[pat].double() + temb.double()
    ref = torch.nn.functional.layer_norm(x, (d,), g.double(), b.double(), 1e-12)
    # one bf16 rounding of values up to a few units, f32 statistics
    assert ((out.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all()


@pytest.mark.parametrize("n,d", [(1, 4), (3, 5), (70, 33), (300, 768), (2, 4096)])
def test_token_init_clears(n, d):
    i32 = dict(dtype=torch.int32, device=DEV)
    active, cnt, el = torch.full((n,), -1, **i32), torch.zeros(1, **i32), torch.zeros(n, **i32)
    guard = torch.full((n * d + 8,), 3.0, device=DEV)
    for off in (4, 1):                  # 16-byte aligned; not
        guard.fill_(3.0)
        B.token_init(n, 7, d, active, cnt, el, guard[off:off + n * d])
        assert int(cnt) == n and torch.equal(active, torch.arange(n, **i32)) and (el == 7).all()
        assert (guard[off:off + n * d] == 0).all()
        assert (guard[:off] == 3).all() and (guard[off + n * d:] == 3).all()


@pytest.mark.parametrize("rows,d", [(1, 64), (5, 320), (7, 4096), (3, 4160)])
def test_final_norm(rows, d):
    """x_norm of the head's RMSNorm (the scratch output) against torch."""
    bf = torch.bfloat16
    h, gain = _rows(rows, d, bf), _rows(1, d, bf, seed=5)[0]
    head = _rows(64, d, bf, seed=6)
    r = torch.arange(rows, dtype=torch.int32, device=DEV)
    xn, logits = torch.empty_like(h), torch.empty((rows, 64), device=DEV)
    n = torch.tensor([rows], dtype=torch.int32, device=DEV)
    B.final_logits(d, 64, 1e-6, h, h, torch.zeros_like(r), r, n, rows, gain, head, xn, logits)
    x = h.double()
    ref = x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6) * gain.double()
    assert ((xn.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-6).all()
    lref = xn.double() @ head.double().T
    assert ((logits.double() - lref).abs().max() <= 2e-6 * d ** 0.5 * lref.abs().max()).all()
