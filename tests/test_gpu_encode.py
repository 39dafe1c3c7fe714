"""Enrollment encodes on the GPU exactly what the client's encoder (fa_encode, on the host) gives
for the same slots: the same float64 butterflies, so the same integers, word for word, in every
layout, at ragged sizes, and for values no encoding holds (which become INT64_MIN)."""
import numpy as np
import pytest

from common import say

pytestmark = pytest.mark.gpu


def context(logn, L, K=1):
    from paper_2608_21131_amd import fa
    return fa, fa.Context(logn, L, K, 40)


def same(ctx, got, slots):
    """got (a Buf of plaintexts) against the host encoder's integers of each slot vector."""
    ref = ctx.encode_db_block_int(np.stack([ctx.encode(v) for v in slots]))
    assert got.count == ref.count
    assert np.array_equal(got.t.cpu().numpy(), ref.t.cpu().numpy())


@pytest.mark.parametrize("logn,L,rows,dim,d,B", [(10, 1, 512, 16, 16, 4), (11, 3, 1000, 7, 8, 8), (12, 2, 1, 1, 128, 16),
                                                 (13, 3, 4095, 100, 128, 32), (14, 1, 5000, 33, 64, 64),
                                                 (15, 3, 16384, 96, 128, 32), (16, 2, 30000, 70, 128, 1)])
def test_diagonal_blocks(logn, L, rows, dim, d, B):
    fa, ctx = context(logn, L)
    X = np.random.default_rng(logn).standard_normal((rows, dim)).astype(np.float32)
    say(f"[encode] N=2^{logn} {rows} x {dim} in {d} diagonals")
    got = ctx.encode_db_block(X, d, fa.LAYOUT_DIAG, B)
    S, slots = ctx.slots, []
    i = np.arange(rows)
    for j in range(d):
        col = (i + j) % d
        v = np.zeros(S)
        v[(i + (j // B) * B) % S] = np.where(col < dim, X[i, np.minimum(col, dim - 1)], 0.0)
        slots.append(v)
    same(ctx, got, slots)


@pytest.mark.parametrize("logn,L,rows,dim,d", [(10, 2, 33, 16, 16), (13, 3, 70, 100, 128), (15, 2, 129, 1, 256)])
def test_row_layout(logn, L, rows, dim, d):
    fa, ctx = context(logn, L)
    X = np.random.default_rng(rows).standard_normal((rows, dim)).astype(np.float32)
    say(f"[encode] N=2^{logn} {rows} x {dim} in rows of {d}")
    per = ctx.slots // d
    pad = np.zeros((-(-rows // per) * per, d))
    pad[:rows, :dim] = X
    same(ctx, ctx.encode_db_block(X, d, fa.LAYOUT_ROW), pad.reshape(-1, per * d))


@pytest.mark.parametrize("logn,d_in,r,B", [(10, 64, 16, 4), (13, 128, 128, 16), (14, 256, 32, 8)])
def test_projection(logn, d_in, r, B):
    _, ctx = context(logn, 2)
    W = np.random.default_rng(d_in).standard_normal((d_in, r)).astype(np.float32)
    say(f"[encode] N=2^{logn} projection {d_in} x {r}")
    s = np.arange(ctx.slots)
    slots = [np.roll(W[(s + j) % d_in, s % r].astype(np.float64), (j // B) * B) for j in range(r)]
    same(ctx, ctx.encode_projection(W, B), slots)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 1e30])
def test_values_without_an_encoding(bad):
    fa, ctx = context(11, 2)
    X = np.zeros((10, 4), dtype=np.float32)
    X[3, 1] = bad
    got = ctx.export(ctx.encode_db_block(X, 4, fa.LAYOUT_DIAG, 2))
    j = (1 - 3) % 4  # the diagonal that holds row 3's column 1, rotated right by its giant step
    v = np.zeros(ctx.slots)
    v[3 + (j // 2) * 2] = np.float32(bad)
    ints = ctx.encode(v)
    assert np.any(ints == np.iinfo(np.int64).min)  # out of range in some coefficients at least
    for t, q in enumerate(ctx.primes[:ctx.L]):
        assert np.array_equal(got[j, t], np.array([int(x) % q for x in ints], dtype=np.uint64))
    assert not got[[k for k in range(4) if k != j]].any()
