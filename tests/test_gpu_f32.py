"""The f32 path on both of its GEMM forms: the matrix-instruction kernel at row
counts around its 16-row tile and at K and N with remainders, and the general
form (rotary heads not a multiple of 32, K not a multiple of 4), free-running
on a fixed exit schedule against the oracle at the f32 bound (1e-5)."""
import math

import numpy as np
import pytest
import torch

import adept_inputs as ai
from oracle import adept_oracle as O
from paper_2601_03700_amd import binding as B
from paper_2601_03700_amd.model import DecoderModel

pytestmark = pytest.mark.gpu

# K of 100 and 132 (part of a 32-deep piece), vocab 100 (part of a 16-column tile)
FUSED = ai.DecoderShape(n_layers=3, d_model=100, n_heads=3, head_dim=32, d_ff=132, vocab=100)
GENERAL = ai.DecoderShape(n_layers=3, d_model=96, n_heads=6, head_dim=16, d_ff=130, vocab=100)


def rel_err(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30))


@pytest.mark.parametrize("shape", [FUSED, GENERAL])
@pytest.mark.parametrize("Bn,T", [(1, 1), (1, 16), (1, 17), (3, 21)])
def test_f32_forms(shape, Bn, T):
    w = ai.decoder_weights(shape, seed=T, dtype="f32", std=0.08)
    ids = ai.token_ids(T, shape.vocab, Bn, T)
    force = np.random.default_rng(T).integers(0, shape.n_layers, size=ids.shape).astype(np.int32)
    ref, cref = O.prefill(O.as64(w), shape, ids, O.ExitConfig(delta=math.inf), s_max=T + 1,
                          force_layer=force)
    model = DecoderModel(shape, w, dtype="f32", rope_max_pos=64)
    cfg = B.exit_cfg(math.inf, shape.n_layers)
    cache = model.new_cache(Bn, T + 1, fill=0.0)
    res, _ = model.prefill(ids, cfg, s_max=T + 1, force_layer=force, logits="all", cache=cache)
    np.testing.assert_array_equal(res.exit_layer.cpu().numpy(), ref.exit_layer)
    assert rel_err(res.logits.cpu().numpy(), ref.logits) <= 1e-5
    # a decode step over the computed and generated K/V, exits at layer 1 and 2
    nxt = np.arange(Bn).astype(np.int32)
    f = (np.arange(Bn) % 3).astype(np.int32)
    st_o = O.decode_step(O.as64(w), shape, cref, nxt, np.full(Bn, T), O.ExitConfig(delta=math.inf),
                         force_layer=f)
    st = model.decode_step(cache, torch.from_numpy(nxt).cuda(),
                           torch.full((Bn,), T, dtype=torch.int32, device="cuda"), cfg,
                           force_layer=torch.from_numpy(f).cuda())
    assert rel_err(st.logits.cpu().numpy(), st_o.logits) <= 1e-5
    k, v = (x.cpu().numpy().astype(np.float64) for x in (cache.k, cache.v))
    assert rel_err(k, cref.k) <= 1e-5 and rel_err(v, cref.v) <= 1e-5


def test_f32_general_form_by_size():
    """1280 rows: the outputs of many 64x64 tiles (QKV 780, O and down projections 260)
    take the general form, gate/up (500) and the head stay on the other, and the norm's
    factor reaches both; against the oracle at the f32 bound."""
    shape = ai.DecoderShape(n_layers=2, d_model=832, n_heads=26, head_dim=32, d_ff=1600, vocab=100)
    w = ai.decoder_weights(shape, seed=5, dtype="f32", std=0.03)
    ids = ai.token_ids(5, shape.vocab, 10, 128)
    force = (np.random.default_rng(5).random(ids.shape) < 0.3).astype(np.int32)
    ref, cref = O.prefill(O.as64(w), shape, ids, O.ExitConfig(delta=math.inf), s_max=128,
                          force_layer=force)
    model = DecoderModel(shape, w, dtype="f32", rope_max_pos=128)
    cache = model.new_cache(10, 128, fill=0.0)
    B.timing_reset()
    B.timing_enable(True)
    res, _ = model.prefill(ids, B.exit_cfg(math.inf, shape.n_layers), s_max=128, force_layer=force,
                           logits="all", cache=cache)
    torch.cuda.synchronize()
    B.timing_enable(False)
    launches = {k: n for k, (n, _) in B.timing_read().items()}
    general = sum(n for k, n in launches.items() if k.startswith("gemm_f32_kernel"))
    fused = sum(n for k, n in launches.items() if "gemm_f32_mfma_kernel" in k)
    print(launches, flush=True)
    assert general == 3 * shape.n_layers   # QKV, O and down projections
    assert fused == shape.n_layers + 2     # gate/up; the K/V generation, the head
    assert rel_err(res.logits.cpu().numpy(), ref.logits) <= 1e-5
    k, v = (x.cpu().numpy().astype(np.float64) for x in (cache.k, cache.v))
    assert rel_err(k, cref.k) <= 1e-5 and rel_err(v, cref.v) <= 1e-5
