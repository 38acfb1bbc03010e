"""The two tile sizes of the grouped K/V generation: few tiles (128x128) and
more than 512 of 256x256, rows at the edges of either, an empty second half of a
256-row item, ragged columns, K of few stages.  Which tile ran is read from the
kernels' names.  Against plain torch in 64 bits; one bf16 rounding of sums with
f32 error, per element."""
import contextlib

import numpy as np
import pytest
import torch

from paper_2601_03700_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _normal(dims, seed, std=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return (torch.randn(dims, generator=g, device=DEV) * std).to(torch.bfloat16)


@contextlib.contextmanager
def _on_tiles(name):
    """The K/V generation inside runs on these tiles."""
    B.timing_reset()
    B.timing_enable(True)
    yield
    torch.cuda.synchronize()
    B.timing_enable(False)
    ran = [n for n in B.timing_read() if "gemm_kv_flat" in n]
    assert ran == [f"gemm_kv_flat_kernel<{name}>"], ran


def _close(got, want, K):
    # the result's bf16 rounding (up to 2^-8 of it) and f32 sums of K products
    # (about K 2^-24 of the result's spread)
    tol = want.abs() * 2.0 ** -8 + K * 2.0 ** -22 * want.std()
    assert ((got.double() - want).abs() <= tol).all()


@pytest.mark.parametrize("layers,rows", [(2, 1), (2, 127), (2, 128), (3, 129), (3, 256), (4, 257),
                                         (40, 385)])
def test_rmsnorm_family(layers, rows):
    with _on_tiles("128x128"):
        _rmsnorm(layers, rows, 320, 4, 64)


# K of 1 to 7 stages: fewer than the five slots of the ring, each remainder past them
@pytest.mark.parametrize("D,rows,hd", [(64, 1025, 64), (128, 1056, 128), (192, 1280, 64),
                                       (256, 1281, 128), (320, 1025, 128), (384, 1100, 64),
                                       (448, 1152, 128)])
def test_rmsnorm_family_many_tiles(D, rows, hd):
    with _on_tiles("256x256"):
        _rmsnorm(64, rows, D, 256 // hd, hd)     # 640 tiles at least


def _rmsnorm(layers, rows, D, H, hd):
    print(f"kv tiles layers={layers} rows={rows} D={D} hd={hd}", flush=True)
    s, w = _normal((rows, D), rows), _normal((layers, 2 * H * hd, D), layers, 0.05)
    el = torch.from_numpy(np.random.default_rng(rows).integers(1, layers + 1, rows).astype(np.int32)).to(DEV)
    idx = torch.arange(rows, dtype=torch.int32, device=DEV)
    n = torch.tensor([rows], dtype=torch.int32, device=DEV)
    cos, sin = (torch.empty((rows, hd // 2), device=DEV) for _ in range(2))
    B.rope_table(rows, hd, 10000.0, cos, sin)
    k, v = (torch.full((layers, rows, H, hd), -9.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = torch.empty(B.kv_generate_workspace_bytes(layers, rows), dtype=torch.uint8, device=DEV)
    B.kv_generate(layers, D, H, hd, 1e-6, s, idx, n, rows, el, idx, idx, w, w.stride(0), None, cos, sin,
                  k, v, rows, ws)
    x = s.double() / torch.sqrt((s.double() ** 2).mean(-1, keepdim=True) + 1e-6)
    c, sn = cos.double()[:, None], sin.double()[:, None]
    for r in range(1, layers + 1):
        on = el < r
        y = (x @ w[r - 1].double().T).view(rows, 2, H, hd)
        a, b = y[:, 0, :, :hd // 2], y[:, 0, :, hd // 2:]
        rot = torch.cat([a * c - b * sn, b * c + a * sn], -1)
        if on.any():
            _close(k[r - 1][on], rot[on], D)
            _close(v[r - 1][on], y[:, 1][on], D)
        assert (k[r - 1][~on] == -9.0).all() and (v[r - 1][~on] == -9.0).all()


@pytest.mark.parametrize("layers,rows", [(2, 128), (3, 200), (3, 257), (40, 300)])
def test_layernorm_family(layers, rows):
    with _on_tiles("128x128"):
        _layernorm(layers, rows, 448)


@pytest.mark.parametrize("D,rows", [(64, 769), (192, 800), (448, 1024)])
def test_layernorm_family_many_tiles(D, rows):
    with _on_tiles("256x256"):
        _layernorm(64, rows, D)


def _layernorm(layers, rows, D):
    H, hd = 5, 64                       # 640 columns: ragged 256-column tiles
    print(f"kv tiles layernorm layers={layers} rows={rows} D={D}", flush=True)
    s, w = _normal((rows, D), rows), _normal((layers, 2 * H * hd, D), layers, 0.05)
    bias = _normal((layers, 2 * H * hd), 7, 0.1)
    el = torch.from_numpy(np.random.default_rng(rows).integers(1, layers + 1, rows).astype(np.int32)).to(DEV)
    idx = torch.arange(rows, dtype=torch.int32, device=DEV)
    n = torch.tensor([rows], dtype=torch.int32, device=DEV)
    k, v = (torch.full((layers, rows, H, hd), -9.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = torch.empty(B.kv_generate_layernorm_workspace_bytes(layers, rows, D), dtype=torch.uint8, device=DEV)
    B.kv_generate_layernorm(layers, D, H, hd, 1e-5, s, idx, n, rows, el, idx, w, w.stride(0), bias,
                            bias.stride(0), k, v, rows, ws)
    # the kernels normalise to bf16 first
    x = torch.nn.functional.layer_norm(s.double(), (D,), eps=1e-5)
    for r in range(1, layers + 1):
        on = el < r
        y = (x @ w[r - 1].double().T + bias[r - 1].double()).view(rows, 2, H, hd)
        for got, want in ((k, y[:, 0]), (v, y[:, 1])):
            if on.any():
                # bf16 keeps 8 bits: rounding moves x by up to 2^-8 |x| (half a step at the
                # low end of a binade), uniform, so by at most 2^-8 / sqrt(3) |x| in the rms;
                # D independent ones times weights of rms 0.05 (x has rms 1), six sigma
                e = (got[r - 1][on].double() - want[on]).abs()
                noise = 6 * 2.0 ** -8 / 3 ** 0.5 * 0.05 * D ** 0.5
                assert (e <= want[on].abs() * 2.0 ** -8 + noise).all()
            assert (got[r - 1][~on] == -9.0).all()
