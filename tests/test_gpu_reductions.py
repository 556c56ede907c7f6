"""GPU parity of the reductions of partial sums: the split-K slices of the
prefill GEMM (with 16-byte accesses where rows and pointers allow them, else
one output at a time) and the column tiles of the version-2 GEMV (16 parts per
output for few outputs, 4 for many).  Bars as for those paths: 1e-4 normwise
against the exact product in fp64.
"""
import numpy as np
import pytest

import oracle
import synth
from gemv_ref import TOL_EXACT, exact_gemv, normwise
from synth.configs import small_spec

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eq():
    import paper_2601_22787_amd as m
    m.lib()
    assert torch.cuda.is_available()
    return m


def make(eq, M, N, version, seed, **kw):
    spec = small_spec(M, N, bits=3.0, chunk=1024, lanes=64, seed=seed)
    w = synth.weights(spec)
    alpha, _ = eq.eqe_alpha_search(w, 3.0)
    if version == 1:
        blob = eq.eqe_encode(w, alpha, chunk_syms=1024, lanes=64)
        rc, q = oracle.container_decode(blob)
    else:
        blob = eq.eqe_encode2(w, alpha, **kw)
        rc, q = oracle.container2_decode(blob)
    assert rc == oracle.OK
    return eq.Layer(blob), q, oracle.container_scales(blob), spec


def spread(spec, B):
    """Activations over 24 binary orders, so that sums in another order differ
    in their last bits."""
    x = synth.activations(spec, B).astype(np.uint32) << 16
    e = np.random.default_rng(spec.seed).integers(-12, 13, x.shape)
    return (np.ldexp(x.view(np.float32), e).view(np.uint32) >> 16).astype(np.uint16)


def device(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("M", [4, 258, 300])
@pytest.mark.parametrize("N", [512, 2560])  # 2 slices; 10 (past two groups of four)
def test_split_sums(eq, M, N, shift):
    print("split sums", M, N, shift, flush=True)
    L, q, s, spec = make(eq, M, N, 1, M + N)
    B = 33
    x = np.stack([synth.vector(spec.seed, 60 + t, N) for t in range(B)])
    bias = synth.bias(spec)
    codes = torch.from_numpy(q.copy()).cuda()
    need = eq.eq_gemm_codes_workspace_bytes(L, B)
    assert need > 0
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")[4 * shift:4 * shift + need]
    y = torch.full((B * M + 4,), float("nan"), dtype=torch.float32, device="cuda")[shift:]
    eq.eq_gemm_codes(L, codes, device(x), B, device(bias), y, ws)
    got = y[:B * M].cpu().numpy().reshape(B, M)
    assert (normwise(got, exact_gemv(q, s, x, bias_bits=bias)) <= TOL_EXACT).all()
    assert np.isnan(y[B * M:].cpu().numpy()).all()


@pytest.mark.parametrize("M,N,TC", [(4096, 68, 4), (4097, 68, 4), (4097, 8, 4), (4100, 24, 8)])
def test_tile_sums(eq, M, N, TC):
    """32768 outputs at batch 8 (the most of 16 parts) and just over."""
    print("tile sums", M, N, TC, flush=True)
    L, q, s, spec = make(eq, M, N, 2, M + N, tile_rows=128, tile_cols=TC)
    x = synth.activations(spec, 8)
    for B in (1, 8):
        y = torch.full((B, M), float("nan"), dtype=torch.float32, device="cuda")
        eq.eq_decode_gemv(L, device(x[:B]), B, None, y, L.workspace(B))
        assert (normwise(y.cpu().numpy(), exact_gemv(q, s, x[:B])) <= TOL_EXACT).all()


@pytest.mark.parametrize("order", [False, True])
def test_joint_tile_sums_as_single(eq, order):
    """A layer's outputs do not depend on the layers it shares a launch with:
    33 column tiles (fifteen parts of 2 tiles and one of 3), one layer with
    more than 32768 outputs, one with fewer and one of a single tile
    height, against each layer's own call."""
    print("joint tile sums", order, flush=True)
    made = [make(eq, M, 132, 2, 500 + M, tile_rows=128, tile_cols=4, row_order=order)
            for M in (4160, 300, 128)]
    layers = [m[0] for m in made]
    x = spread(made[0][3], 8)
    for B in (5, 8):
        ys = [torch.full((B, L.rows), float("nan"), dtype=torch.float32, device="cuda")
              for L in layers]
        eq.eq_decode_gemv_multi(layers, device(x[:B]), B, None, ys, eq.multi_workspace(layers, B))
        for (L, q, s, _), y in zip(made, ys):
            one = torch.full((B, L.rows), float("nan"), dtype=torch.float32, device="cuda")
            eq.eq_decode_gemv(L, device(x[:B]), B, None, one, L.workspace(B))
            assert torch.equal(y, one), (L.rows, B)
            assert (normwise(y.cpu().numpy(), exact_gemv(q, s, x[:B])) <= TOL_EXACT).all()


def test_tile_sums_do_not_depend_on_the_batch(eq):
    """A token's outputs beside four others (23500 outputs, below the change of
    the number of wavefronts per output) and beside seven (37600, above)."""
    print("batch", flush=True)
    L, q, s, spec = make(eq, 4700, 132, 2, 9, tile_rows=128, tile_cols=4)
    x = spread(spec, 8)
    ys = []
    for B in (5, 8):
        y = torch.full((B, L.rows), float("nan"), dtype=torch.float32, device="cuda")
        eq.eq_decode_gemv(L, device(x[:B]), B, None, y, L.workspace(B))
        ys.append(y)
    assert torch.equal(ys[0], ys[1][:5])
