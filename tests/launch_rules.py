"""The library's launch rules in Python (a helper module of the tests, not a
test file), so that a test can name the path its shape is meant for.
tests/test_launch_rules.py holds them to the C++ of csrc/eq_rules.h."""

CUS = 256  # compute units of an MI355X


def ragged_fused(n_chunks, cols, chunk_syms, B, cus=CUS):
    t = 1.0 if B == 1 else 1.25 if B == 2 else 2.0 if B <= 4 else 3.0
    return (n_chunks * (1.0 + B * cols / 8192.0) >= t * cus or
            cols >= (0.25 if B == 1 else 0.4) * chunk_syms)


def v1_gemv_route(M, N, C, lanes, B):
    """How a version-1 GEMV whose rows are not whole steps runs: 'cols' (fused,
    over transposed activations) or 'codes' (over the decoded codes)."""
    assert N % lanes
    nc = -(-M * N // C)
    part = -(-8 * nc * B // 256) * 256
    xc = 0 if B == 1 else N * (4 if B == 2 else 8 if B <= 4 else 16)
    fits = part + xc + 3 <= -(-M * N // 256) * 256
    return "cols" if N >= 64 and fits and ragged_fused(nc, N, C, B) else "codes"
