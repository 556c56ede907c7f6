"""GPU parity of the version-1 GEMV over transposed activations: 64 lanes, and
rows that are not whole steps, and the GEMV over decoded codes.

Shapes sit at the edges of its units (128 columns at 64 and 128 lanes, 256 at
256 lanes): rows shorter than a unit, rows that end inside one, at its end or
inside its first 64 columns, rows longer than a chunk, a whole step past the
last unit, a partial last step.  The bars are those of the fused GEMV: 1e-4
normwise against the exact product in fp64 (fp32 accumulation of up to 4160
terms is a few 1e-6; one wrong term shows at about 1e-3).
"""
import numpy as np
import pytest

import launch_rules
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


def make(eq, M, N, C, lanes, fmt, seed):
    spec = small_spec(M, N, bits=3.0, chunk=C, lanes=lanes, seed=seed)
    w = synth.weights(spec)
    alpha, _ = eq.eqe_alpha_search(w, 3.0, base_format=fmt)
    blob = eq.eqe_encode(w, alpha, chunk_syms=C, lanes=lanes, base_format=fmt)
    rc, q = oracle.container_decode(blob)
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


def gemv(eq, L, x_bits, bias_bits=None, ws=None):
    B = x_bits.shape[0]
    y = torch.full((B, L.rows), float("nan"), dtype=torch.float32, device="cuda")
    eq.eq_decode_gemv(L, device(x_bits), B, None if bias_bits is None else device(bias_bits), y,
                      L.workspace(B) if ws is None else ws)
    return y.cpu().numpy()


SHAPES = [
    # M, N, C, lanes
    (70, 64, 256, 64),      # a row per sub-step, two rows per unit
    (9, 192, 320, 64),      # rows end inside units; five steps per chunk (one past the units)
    (33, 128, 128, 64),     # a row per unit, a chunk per row
    (5, 4160, 2048, 64),    # rows longer than chunks
    # ragged
    (200, 65, 128, 64),     # one lane past the row's end
    (60, 127, 256, 128),    # just under a unit
    (60, 129, 256, 128),    # just over
    (64, 333, 512, 256),    # rows of a unit and part of one
    (120, 110, 256, 256),   # rows shorter than a unit
    (64, 1001, 256, 64),    # rows over several chunks, partial last step
    (6000, 100, 768, 256),  # many short rows in many chunks
    (24, 4161, 2048, 256),  # long rows at 256 lanes
]
# ragged, but decoded to codes first: under 64 columns; workspaces too small
# for the transposed activations; few chunks that hold many rows
CODES = [(50, 63, 256, 64, 1), (50, 63, 256, 64, 8), (2, 70, 64, 64, 8), (7, 100, 256, 256, 8),
         (64, 333, 1024, 256, 3), (500, 100, 4096, 128, 1), (13, 333, 4096, 256, 8)]


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("M,N,C,lanes", SHAPES)
def test_shapes(eq, M, N, C, lanes, fmt):
    print("gemv over columns", M, N, C, lanes, fmt, flush=True)
    L, q, s, spec = make(eq, M, N, C, lanes, fmt, 7 * M + N)
    bias = synth.bias(spec)
    for B in (1, 2, 3, 5, 8):
        assert N % lanes == 0 or launch_rules.v1_gemv_route(M, N, C, lanes, B) == "cols"
        x = synth.activations(spec, B)
        y = gemv(eq, L, x, bias)
        err = normwise(y, exact_gemv(q, s, x, fmt=fmt, bias_bits=bias))
        assert (err <= TOL_EXACT).all(), (B, err)
    assert eq.eq_get_status(L) == eq.EQ_OK


@pytest.mark.parametrize("M,N,C,lanes,B", CODES)
def test_shapes_over_codes(eq, M, N, C, lanes, B):
    print("gemv over codes", M, N, C, lanes, B, flush=True)
    assert launch_rules.v1_gemv_route(M, N, C, lanes, B) == "codes"
    L, q, s, spec = make(eq, M, N, C, lanes, 1, 7 * M + N)
    bias = synth.bias(spec)
    x = synth.activations(spec, B)
    err = normwise(gemv(eq, L, x, bias), exact_gemv(q, s, x, bias_bits=bias))
    assert (err <= TOL_EXACT).all(), err
    assert eq.eq_get_status(L) == eq.EQ_OK


def test_infinity_stays_in_its_row(eq):
    """A batch row with an infinite activation leaves the other rows as they are."""
    print("infinity", flush=True)
    L, q, s, spec = make(eq, 40, 449, 1024, 64, 1, 3)
    assert launch_rules.v1_gemv_route(40, 449, 1024, 64, 8) == "cols"
    x = synth.activations(spec, 8)
    y = gemv(eq, L, x)
    assert (normwise(y, exact_gemv(q, s, x)) <= TOL_EXACT).all()
    x2 = x.copy()
    x2[3, 17] = x2[3, 448] = 0x7F80
    y2 = gemv(eq, L, x2)
    keep = [b for b in range(8) if b != 3]
    assert np.array_equal(y2[keep], y[keep])
    assert not np.isfinite(y2[3]).all()


@pytest.mark.parametrize("lanes", [64, 128])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 8])
def test_joint_launch(eq, B, lanes):
    """Layers of one or two states per lane that share an input: one launch,
    the single calls' bits."""
    print("joint", lanes, "lanes", B, flush=True)
    made = [make(eq, M, 7 * lanes, 1024, lanes, 1, 50 + M) for M in (65, 8, 130)]
    layers = [m[0] for m in made]
    x = synth.activations(made[0][3], B)
    ys = [torch.full((B, L.rows), float("nan"), dtype=torch.float32, device="cuda")
          for L in layers]
    eq.eq_decode_gemv_multi(layers, device(x), B, None, ys, eq.multi_workspace(layers, B))
    for (L, q, s, _), y in zip(made, ys):
        y = y.cpu().numpy()
        assert np.array_equal(y, gemv(eq, L, x))
        assert (normwise(y, exact_gemv(q, s, x)) <= TOL_EXACT).all()


@pytest.mark.parametrize("M,N,C,lanes,shift", [
    (40, 448, 1024, 64, 4), (33, 128, 128, 64, 4),               # whole rows of steps
    (64, 333, 512, 256, 4), (64, 1001, 1024, 64, 4), (64, 1001, 1024, 64, 1),
    (50, 63, 256, 64, 1),                                        # over the decoded codes
])
def test_workspace_address(eq, M, N, C, lanes, shift):
    """Where the workspace lies (4-byte aligned; at any byte for rows that are
    not whole steps) does not change a bit, alone and in a joint call."""
    print("workspace address", M, N, C, lanes, shift, flush=True)
    L, q, s, spec = make(eq, M, N, C, lanes, 1, M + N)
    for B in (1, 2, 3, 8):
        x = spread(spec, B)
        y = gemv(eq, L, x)
        assert (normwise(y, exact_gemv(q, s, x)) <= TOL_EXACT).all()
        room = torch.empty(L.workspace(B).numel() + 16, dtype=torch.uint8, device="cuda")
        at = room[shift:shift + L.workspace(B).numel()]
        assert np.array_equal(gemv(eq, L, x, ws=at), y), B
        room = torch.empty(eq.eq_gemv_multi_workspace_bytes([L, L], B) + 16, dtype=torch.uint8,
                           device="cuda")
        ys = [torch.full((B, M), float("nan"), dtype=torch.float32, device="cuda")
              for _ in range(2)]
        eq.eq_decode_gemv_multi([L, L], device(x), B, None, ys, room[shift:])
        assert all(np.array_equal(t.cpu().numpy(), y) for t in ys), B


@pytest.mark.parametrize("M,N,C", [(8, 64, 64), (95, 2112, 4096)])
def test_batch1_input_address(eq, M, N, C):
    """64 lanes at batch 1: the input staged 16 bytes at a time where it is
    16-byte aligned, value by value where it is not; the same bits."""
    print("batch-1 input address", M, N, C, flush=True)
    L, q, s, spec = make(eq, M, N, C, 64, 1, M + N)
    x = spread(spec, 1)
    y = gemv(eq, L, x)
    assert (normwise(y, exact_gemv(q, s, x)) <= TOL_EXACT).all()
    room = torch.empty(N + 8, dtype=torch.int16, device="cuda")
    for shift in (1, 4):
        room[shift:shift + N] = device(x)[0]
        y2 = torch.full((1, M), float("nan"), dtype=torch.float32, device="cuda")
        eq.eq_decode_gemv(L, room[shift:shift + N], 1, None, y2, L.workspace(1))
        assert np.array_equal(y2.cpu().numpy(), y)
