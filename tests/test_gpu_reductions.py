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
