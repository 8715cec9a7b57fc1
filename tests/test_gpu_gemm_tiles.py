"""GPU parity of the dense pass over the GEMM's tile configs and split counts.

One-layer models whose row counts and widths make the plan pick every tile config for every
epilogue of the layers, whole-K and split-K (test_gemm_plan.py checks that they do), with
remainders in rows (a last tile of 1 to 130 rows), columns (ffn and head widths that are no
multiple of the tile) and K (1 to 256 slices of 32), and batches whose sequences straddle the row
tiles and the runs of 8 positions in which v is written, or of which several share a wavefront's
rows.
Oracle: oracle.forward in fp64; bound: the one of the other forward tests, 2e-2 x max |logit|.
"""
import numpy as np
import pytest

import seeded_inputs as si
import tests.test_gpu_lm_head as lmh
from oracle import forward as of
from tests.gpu_common import log_case, require_gpu, to_dev
from tests.parity import bf16_to_f32, logit_tolerance

pytestmark = pytest.mark.gpu

# (batch, length), d, heads, kv heads, head dim, ffn
SHAPES = [
    ((1, 1), 64, 1, 1, 64, 64),            # one row, one slice pair
    ((1, 97), 512, 8, 2, 64, 688),         # 32 x 64 tiles; O split 2
    ((2, 65), 1024, 8, 2, 128, 2816),      # O, down split 4
    ((4, 65), 1024, 8, 2, 128, 2816),      # 64 x 64 and 64 x 128 tiles
    ((13, 79), 512, 8, 8, 64, 4000),       # 256 x 192 gate/up, 128 x 64 QKV, odd rows
    ((4, 500), 512, 4, 4, 128, 12288),     # 256 x 256 gate/up
    ((4, 500), 512, 32, 32, 128, 4032),    # 256 x 192 QKV
    ((1, 513), 2048, 4, 1, 64, 8192),      # 192 x 128 gate/up and down (split 4)
    ((3, 333), 2048, 16, 16, 128, 1100),   # 128 x 192 QKV
    ((1, 65), 4096, 4, 2, 128, 1024),      # QKV split 8: partials and their finish kernel
    ((4, 65), 8192, 4, 2, 128, 64),        # widest d, 256 slices
    ((8, 375), 256, 16, 16, 128, 1200),    # many row tiles (more than one group of 8)
    ((4, 575), 256, 32, 16, 64, 640),
    ((6, 215), 1024, 32, 32, 128, 512),    # 192 x 128 QKV and O, 138 rows in the last tile
    ((3, 1000), 1024, 24, 24, 128, 512),
    ((1, 700), 512, 24, 24, 128, 128),     # 256 x 128 QKV, last tile of 188 rows
    # three sequences or more in the rows of one wavefront (16, 32, 64 and 96)
    ((40, 1), 256, 4, 4, 64, 64),
    ((70, 2), 256, 16, 16, 128, 64),
    ((64, 10), 512, 4, 2, 128, 64),
    ((64, 20), 512, 4, 4, 64, 64),
    ((50, 40), 512, 16, 16, 128, 64),
    ((12, 39), 256, 64, 1, 128, 64),
    # the configs of each epilogue that the shapes above leave out
    ((8, 163), 3008, 8, 2, 128, 146),      # QKV and down 64 x 128, O 192 x 128
    ((8, 243), 7424, 4, 4, 64, 36),        # QKV split 4, 128 x 192; O 256 x 256
    ((4, 400), 6400, 4, 2, 128, 64),       # QKV split 4, 256 x 128; O 256 x 192
    ((4, 875), 1984, 1, 1, 128, 889),      # down and gate/up 256 x 128
    ((1, 1930), 448, 1, 1, 64, 1476),      # gate/up 128 x 192
    ((8, 296), 2496, 8, 2, 64, 60),        # O 128 x 192
    ((8, 165), 384, 80, 4, 64, 66),        # O split 4, 64 x 128
    ((5, 41), 6400, 24, 24, 128, 64),      # QKV split 4, 256 x 192
    ((3, 258), 3520, 100, 4, 128, 64),     # O split 4, 256 x 256
]


@pytest.mark.parametrize("bl,d,H,Hkv,hd,ffn", SHAPES, ids=lambda v: str(v).replace(" ", ""))
def test_one_layer(bl, d, H, Hkv, hd, ffn):
    require_gpu()
    from paper_2608_11235_amd import Model
    B, L = bl
    spec = si.ModelSpec("tiles", 1, d, H, Hkv, hd, ffn, 500, 7, True, 1e-6, 1e6, 6.0)
    log_case(f"tiles B={B} L={L} d={d} H={H}/{Hkv}x{hd} ffn={ffn}")
    tokens = si.prompt_tokens(3, B, L, spec.vocab, spec.mask_id)
    rows = np.unique(np.concatenate([np.arange(min(L, 12)), np.arange(max(0, L - 12), L)]))
    with Model(spec, seed=1, max_batch=B, max_seq=L) as m:
        got = bf16_to_f32(m.forward_logits(to_dev(tokens), 0, L).cpu().numpy())[:, rows]
    ref = of.forward_logits(si.HostWeights(spec, 1), spec, tokens, rows)
    err = np.abs(got.astype(np.float64) - ref)
    print(f"max_err={err.max():.4g} tol={logit_tolerance(ref):.4g}")
    assert err.max() <= logit_tolerance(ref)


# rows and vocabularies (no multiples of 32, so the last weight group and tile are ragged) of the
# tiled LM head: all configs but 256 x 128 and 128 x 192, which HEAD_BLOCKS below has too
HEADS = [(200, 50257), (500, 20011), (500, 9999), (300, 20011), (200, 5003), (130, 20011),
         (130, 5003), (96, 5003), (65, 1001)]


@pytest.mark.parametrize("rows,vocab", HEADS)
def test_tiled_lm_head(rows, vocab):
    require_gpu()
    from paper_2608_11235_amd import Model
    spec = si.ModelSpec("heads", 0, 256, 4, 4, 64, 64, vocab, 7, False, 1e-6, 1e4, 6.0)
    log_case(f"tiled LM head rows={rows} vocab={vocab}")
    tokens = si.prompt_tokens(3, 1, rows, spec.vocab, spec.mask_id)
    with Model(spec, seed=1, max_batch=1, max_seq=rows) as m:
        got = bf16_to_f32(m.forward_logits(to_dev(tokens), 0, rows).cpu().numpy())
    ref = of.forward_logits(si.HostWeights(spec, 1), spec, tokens, np.arange(rows))
    err = np.abs(got.astype(np.float64) - ref)
    print(f"max_err={err.max():.4g} tol={logit_tolerance(ref):.4g}")
    assert err.max() <= logit_tolerance(ref)


# (batch, rows of a block, vocabulary) that take the LM head's logits and its fused scores through
# every tile config at d = 384; the first one's last tile column holds 75 valid columns, so that a
# wavefront column range lies entirely past the vocabulary
HEAD_BLOCKS = [(1, 129, 49227), (2, 66, 43875), (3, 129, 12385), (1, 68, 33071), (1, 65, 16913),
               (1, 66, 10907), (2, 65, 8223), (1, 65, 5465), (1, 65, 525), (1, 129, 21787)]


@pytest.mark.parametrize("B,blk,vocab", HEAD_BLOCKS)
def test_tiled_lm_head_and_scores(B, blk, vocab):
    """Logits against the oracle, and the fused scores against the logits' own."""
    require_gpu()
    from paper_2608_11235_amd import Model
    spec = si.ModelSpec("heads", 0, 384, 6, 6, 64, 64, vocab, 7, False, 1e-6, 1e4, 6.0)
    log_case(f"tiled LM head and scores B={B} blk={blk} vocab={vocab}")
    tokens = si.prompt_tokens(3, B, blk, spec.vocab, spec.mask_id)
    with Model(spec, seed=1, max_batch=B, max_seq=blk) as m:
        got = bf16_to_f32(m.forward_logits(to_dev(tokens), 0, blk).cpu().numpy())
    ref = of.forward_logits(si.HostWeights(spec, 1), spec, tokens, np.arange(blk))
    err = np.abs(got.astype(np.float64) - ref)
    print(f"max_err={err.max():.4g} tol={logit_tolerance(ref):.4g}")
    assert err.max() <= logit_tolerance(ref)
    lmh.test_fused_scores_match_own_logits(spec, B, blk)
