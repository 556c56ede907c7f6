"""GPU parity of version-2 codes and BF16 output around its segment length.

A launch writes whole segments of 32 or 64 codes, chosen from the tile widths
and heights, with a smaller stream window and shorter list entries for 64-code
segments of 256-row tiles.  The shapes sit at the edges: tile rows shorter than
a segment, exactly one, one and a partial one; tile rows of as many segments as
a list entry can number, and more; layers of several heights in one launch.
Decoding is lossless, so every output equals the oracle's.
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from synth.configs import small_spec

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eq():
    import paper_2601_22787_amd as m
    m.lib()
    assert torch.cuda.is_available()
    return m


def make(eq, M, N, TR, TC, seed, order=False):
    spec = small_spec(M, N, bits=2.5, seed=seed)
    w = synth.weights(spec)
    alpha, _ = eq.eqe_alpha_search(w, 2.5)
    blob = eq.eqe_encode2(w, alpha, tile_rows=TR, tile_cols=TC, row_order=order)
    rc, q = oracle.container2_decode(blob)
    assert rc == oracle.OK
    return eq.Layer(blob), q, oracle.dequant(q, oracle.container_scales(blob))


def check(eq, made):
    layers = [m[0] for m in made]
    codes = [torch.full((L.rows, L.cols), 255, dtype=torch.uint8, device="cuda") for L in layers]
    w = [torch.full((L.rows, L.cols), -1, dtype=torch.int16, device="cuda") for L in layers]
    if len(layers) > 1:
        eq.eq_decode_codes_multi(layers, codes)
        eq.eq_decode_bf16_multi(layers, w)
    else:
        eq.eq_decode_codes(layers[0], codes[0])
        eq.eq_decode_bf16(layers[0], w[0])
    for (L, q, ref), c, b in zip(made, codes, w):
        assert np.array_equal(c.cpu().numpy(), q)
        assert np.array_equal(b.cpu().numpy().view(np.uint16), ref)
        assert eq.eq_get_status(L) == eq.EQ_OK


@pytest.mark.parametrize("order", [False, True])
@pytest.mark.parametrize("TR,M", [(64, 70), (128, 150), (256, 300)])
@pytest.mark.parametrize("TC,N", [(60, 200), (64, 130), (96, 301), (256, 515)])
def test_tile_widths(eq, TR, M, TC, N, order):
    print("segments", TR, TC, M, N, order, flush=True)
    check(eq, [make(eq, M, N, TR, TC, M + N, order)])


@pytest.mark.parametrize("TC", [16384, 16388])
def test_most_segments(eq, TC):
    print("most segments", TC, flush=True)
    check(eq, [make(eq, 257, 16500, 256, TC, TC)])


def test_heights_together(eq):
    print("heights together", flush=True)
    check(eq, [make(eq, 300, 520, 256, 256, 1), make(eq, 130, 260, 128, 128, 2),
               make(eq, 65, 100, 64, 32, 3)])
