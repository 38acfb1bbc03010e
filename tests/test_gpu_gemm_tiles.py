"""The GEMM tiles between the skinny path (at most 64 rows) and the 256-row
tile: row counts at the edges of the 128-row tiles, column counts that leave
ragged 128- and 256-column tiles, and shapes whose tiles are cut along K for each
epilogue of the decoder layer and both tile widths (read from the names of the
reduction kernels).  Whole layers with exits, each checked on the GPU's own inputs against the
oracle (tests/layer_check.py: per element within max(2e-2, one bf16 ulp))."""
import math
import sys

import numpy as np
import pytest
import torch

import adept_inputs as ai
from oracle import adept_oracle as O
from paper_2601_03700_amd import binding as B
from paper_2601_03700_amd.model import DecoderModel, EncoderModel
from tests import layer_check as LC

pytestmark = pytest.mark.gpu

# K of 12 to 26 stages of 64 (the residual GEMM of 26 is cut); N of 13 x 64 and 13 x 128 columns
LLAMA = ai.DecoderShape(n_layers=2, d_model=768, n_heads=6, head_dim=128, d_ff=1664, vocab=384)
GPT2 = ai.DecoderShape(n_layers=2, d_model=832, n_heads=13, head_dim=64, d_ff=1664, vocab=448,
                       family="gpt2", max_pos=512)
ENC = ai.EncoderShape(n_layers=2, d_model=768, n_heads=12, head_dim=64, d_ff=1600, vocab=500,
                      max_pos=512)


# cut tiles: 128 columns (both head sizes; three of the four GEMMs or all), 256 columns
# (SwiGLU, rotary QKV, tanh GELU; the residual one at 128)
CUT_1536 = ai.DecoderShape(n_layers=2, d_model=1536, n_heads=12, head_dim=128, d_ff=3072, vocab=128)
CUT_1280 = ai.DecoderShape(n_layers=2, d_model=1280, n_heads=20, head_dim=64, d_ff=1280, vocab=128)
CUT_GPT2 = ai.DecoderShape(n_layers=2, d_model=1152, n_heads=18, head_dim=64, d_ff=2304, vocab=128,
                           family="gpt2", max_pos=512)
CUT_SWIGLU = ai.DecoderShape(n_layers=1, d_model=3712, n_heads=29, head_dim=128, d_ff=7424, vocab=128)
CUT_QKV = ai.DecoderShape(n_layers=1, d_model=3840, n_heads=30, head_dim=128, d_ff=256, vocab=128)
CUT_GELU = ai.DecoderShape(n_layers=1, d_model=3712, n_heads=58, head_dim=64, d_ff=14848, vocab=128,
                           family="gpt2", max_pos=512)


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("shape,rows", [(LLAMA, 65), (LLAMA, 128), (LLAMA, 129), (LLAMA, 257),
                                        (LLAMA, 385), (GPT2, 65), (GPT2, 127), (GPT2, 300)])
def test_decoder_rows(shape, rows):
    _decoder(shape, rows)


@pytest.mark.parametrize("shape,rows,cut", [
    (CUT_1536, 65, {"qkv_128", "resid_128", "swiglu_128"}),
    (CUT_1536, 128, {"qkv_128", "resid_128", "swiglu_128"}),
    (CUT_1280, 65, {"qkv_128", "resid_128"}),
    (CUT_GPT2, 65, {"qkv_128", "resid_128", "gelu_tanh_128"}),
    (CUT_GPT2, 128, {"qkv_128", "resid_128", "gelu_tanh_128"}),
    (CUT_SWIGLU, 129, {"swiglu_256", "resid_128"}),
    (CUT_QKV, 641, {"qkv_256"}),
    (CUT_GELU, 129, {"gelu_tanh_256", "resid_128"})])
def test_cut_tiles(shape, rows, cut):
    B.timing_reset()
    B.timing_enable(True)
    _decoder(shape, rows)
    torch.cuda.synchronize()
    B.timing_enable(False)
    ran = {n[len("mid_reduce_"):] for n in B.timing_read() if n.startswith("mid_reduce_")}
    say(f"cut: {sorted(ran)}")
    assert cut <= ran


def _decoder(shape, rows):
    say(f"gemm tiles {shape.family} width={shape.d_model} rows={rows}")
    make = ai.gpt2_weights if shape.family == "gpt2" else ai.decoder_weights
    w32 = make(shape, seed=rows, dtype="bf16")
    ids = ai.token_ids(rows, shape.vocab, 1, rows)
    # a third of the rows leave after layer 1: layer 2 has fewer row tiles than
    # the grid, and the K/V of those rows are generated
    force = (np.random.default_rng(rows).random(ids.shape) < 0.34).astype(np.int32)
    model = DecoderModel(shape, w32, dtype="bf16", rope_max_pos=max(512, rows))
    rep = LC.Report(say)
    chk = LC.DecoderLayerCheck(O.as64(w32), shape, None, O.ExitConfig(delta=math.inf), "bf16",
                               force_layer=force, report=rep)
    chk.cache = model.new_cache(1, rows)
    res, _ = model.prefill(ids, B.exit_cfg(math.inf, shape.n_layers), force_layer=force,
                           cache=chk.cache, on_layer=chk)
    chk.finish(res.state, res.logits, res.rows)
    rep.summary()


@pytest.mark.parametrize("rows", [70, 128, 300])
def test_encoder_rows(rows):
    say(f"gemm tiles encoder rows={rows}")
    w32 = ai.encoder_weights(ENC, seed=rows, dtype="bf16")
    ids = ai.token_ids(rows, ENC.vocab, 1, rows)
    force = (np.random.default_rng(rows).random(ids.shape) < 0.34).astype(np.int32)
    force[:, 0] = 0
    rep = LC.Report(say)
    chk = LC.EncoderLayerCheck(O.as64(w32), ENC, O.ExitConfig(delta=math.inf), force_layer=force,
                               report=rep, stop_at_cls=True)
    out = EncoderModel(ENC, w32).classify(ids, B.exit_cfg(math.inf, ENC.n_layers),
                                          force_layer=force, on_layer=chk)
    chk.finish(out, rows)
    rep.summary()


@pytest.mark.parametrize("rows", [3, 30, 64, 65, 200])
def test_rotary_tables_need_no_alignment(rows):
    """Tables that start one float past a 16-byte boundary: the same bits."""
    say(f"gemm tiles unaligned rotary tables rows={rows}")
    shape = ai.DecoderShape(n_layers=1, d_model=1152, n_heads=9, head_dim=128, d_ff=384, vocab=128)
    model = DecoderModel(shape, ai.decoder_weights(shape, seed=1, dtype="bf16"), dtype="bf16",
                         rope_max_pos=512)
    ids = ai.token_ids(rows, shape.vocab, 1, rows)
    caches = []
    for off in (0, 1):
        if off:
            for k in ("rope_cos", "rope_sin"):
                t = getattr(model, k)
                flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
                flat[1:] = t.flatten()
                setattr(model, k, flat[1:].view(t.shape))
        cache = model.new_cache(1, rows)
        model.prefill(ids, B.exit_cfg(math.inf, 1), cache=cache)
        caches.append(cache)
    assert torch.equal(caches[0].k, caches[1].k) and torch.equal(caches[0].v, caches[1].v)
