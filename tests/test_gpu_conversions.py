"""The fused basis conversions of rings from N = 2^14 (ModUp, ModDown and rescale: the column pass
of the inverse transform, the conversion and the first forward pass in one kernel): every column
height, every digit width, short last digits, and launches with the targets in one and in several
groups, each against the oracle word for word."""
import numpy as np
import pytest

import common
from common import Pair, say
from oracle import ckks
from paper_2608_21131_amd import gen

pytestmark = pytest.mark.gpu

SETS = [(14, 3, 1), (14, 5, 2), (14, 2, 3), (15, 4, 3), (15, 3, 4), (15, 2, 1), (16, 2, 1), (16, 3, 2), (16, 5, 4)]
common.PARAMS.update({f"c{logn}_{L}_{K}": (logn, L, K) for logn, L, K in SETS + [(14, 6, 1)]})


# one ciphertext: the targets split into groups; three or five: fewer groups, then one
@pytest.mark.parametrize("logn,L,K,count", [(*s, c) for s in SETS for c in (1, 3)] + [(14, 5, 2, 17), (15, 4, 3, 5)])
def test_rotation_sums(logn, L, K, count):
    p = Pair(f"c{logn}_{L}_{K}", wid=70)
    g = np.random.default_rng(logn + L)
    keys = p.keys([3])
    both = [p.encrypt_both(ckks.encode(g.uniform(-1, 1, p.par.slots), p.n, 40), tag=j) for j in range(count)]
    cts = p.ctx.new_ct(count, log_scale=40)
    for j, (dev, _) in enumerate(both):
        cts.t[j * p.ctx.ct_words:(j + 1) * p.ctx.ct_words] = dev.t
    say(f"[conv] N=2^{logn} {L}+{K} primes, {count} ciphertexts")
    p.ctx.rotate_sum(cts, None, 3, 1)
    got = p.export_ct(cts, count)
    for j in {0, count - 1}:
        assert np.array_equal(got[j], p.orc.rotate_sum(both[j][1], 3, 1, keys)), j


@pytest.mark.parametrize("logn,L", [(11, 2), (13, 4), (14, 2), (14, 6), (15, 5), (16, 2), (16, 4)])
@pytest.mark.parametrize("n_polys", [1, 2, 3])
def test_rescale(logn, L, n_polys):
    from paper_2608_21131_amd import fa
    par = ckks.Params(logn=logn, L=L, K=1)
    hi = fa.Context(logn, L, 1, 40)
    lo = hi.at_level(L - 1)
    x = np.stack([gen.uniform_residues(gen.rng(71, gen.STREAM_ENC_A, h), par.q, 1, par.n)[0] for h in range(n_polys)])
    # the rounding's edges: the last residue 0, either side of half its prime, and its largest
    last = par.q[-1]
    x[:, -1, :4] = [0, (last - 1) // 2, (last + 1) // 2, last - 1]
    say(f"[rescale] N=2^{logn} {L} primes, {n_polys} polynomials")
    buf = hi.import_coeffs(x, n_polys=n_polys)
    got = lo.export(hi.rescale(lo, buf, n_polys=n_polys)).reshape(n_polys, L - 1, par.n)
    assert np.array_equal(got, ckks.Oracle(par).rescale(x))


def giant_groups(logn, L, K, ng, nb):
    """Groups the giants of one launch are split into on two lanes, as the library's rule has them: the
    chip's 512 workgroup places, the sums' scratch (one part per group after the first, in the
    row-passed c1 of the ModUps), the giants and eight bound them; more than 32 giants are not split."""
    np_, n = L + K, 1 << logn
    if ng > 32:
        return 1
    parts = 2 * max(nb, ng) * L * n // (nb * 2 * np_ * n)
    g = max(1, min(512 // ((n >> 12) * np_ * nb), 1 + parts, ng, 8))
    per = -(-ng // g)
    return -(-ng // per)


# giant sums by the groups they are split into: one giant a group (3 and 7 giants, six digits in the
# latter), the cap of eight groups with a short last one (15 and 31), 7 giants in four and in three groups,
# two blocks, splits at N = 2^16, and one group: a single giant, 63 giants (two launches, the second adding
# to the first), so many blocks that the scratch holds no part (6, 9)
@pytest.mark.parametrize("logn,L,K,d,B,blocks,groups", [
    (14, 3, 1, 16, 4, 1, 3), (14, 6, 1, 16, 2, 1, 7), (14, 3, 1, 16, 1, 1, 8), (14, 3, 1, 32, 1, 1, 8),
    (14, 3, 1, 16, 2, 1, 4), (14, 3, 1, 16, 2, 2, 3), (15, 3, 4, 32, 4, 2, 2), (16, 2, 1, 16, 2, 1, 4),
    (16, 2, 1, 32, 2, 1, 8), (16, 2, 1, 8, 4, 1, 1), (14, 5, 2, 64, 1, 1, 1), (14, 5, 2, 16, 2, 6, 1),
    (14, 2, 3, 8, 1, 9, 1)])
def test_split_giant_sums(logn, L, K, d, B, blocks, groups):
    assert giant_groups(logn, L, K, d // B - 1, blocks) == groups
    p = Pair(f"c{logn}_{L}_{K}", wid=72)
    g = np.random.default_rng(d + blocks)
    keys = p.keys(ckks.steps_for_bsgs(d, B))
    ct_dev, ct_orc = p.encrypt_both(ckks.encode(g.uniform(-1, 1, p.par.slots), p.n, 40))
    coeffs = g.integers(-2 ** 30, 2 ** 30, (blocks, d, p.n))
    say(f"[giant] N=2^{logn} {L}+{K} primes d={d} B={B} blocks={blocks}")
    got = p.export_ct(p.ctx.score_block(ct_dev, [p.ctx.encode_db_block_int(c) for c in coeffs], d, 1, B), blocks)
    rots = p.orc.baby_rotations(ct_orc, B, keys)
    for j in {0, blocks - 1}:
        pts = np.stack([ckks.to_residues(c, p.par.q) for c in coeffs[j]]).reshape(d // B, B, p.par.L, p.n)
        assert np.array_equal(got[j], p.orc.bsgs_block(rots, pts, B, d // B, keys)), j
