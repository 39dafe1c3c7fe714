"""Rings up to N = 2^13, whose transforms run one limb (or a quarter of one) per workgroup: the
launch shapes either side of every switch between the fused, quartered and plain kernels, each
against the oracle word for word."""
import numpy as np
import pytest

import common
from common import Pair, say
from oracle import ckks

pytestmark = pytest.mark.gpu

common.PARAMS.update({f"r{logn}_{L}_{K}": (logn, L, K) for logn, L, K in [
    (10, 8, 1), (10, 2, 1), (10, 6, 4), (11, 3, 1), (11, 7, 3), (12, 5, 2), (12, 4, 1), (13, 3, 1), (13, 5, 4)]})


def pair(name, wid):
    return Pair(name, wid=wid)


# (8, 1): a ModUp takes 64 workgroups per ciphertext (quartered to 2, fused to 4, plain from 5) and a
# finish 16 (quartered to 8, fused to 16); 17 ciphertexts are two batches.  Odd and even step counts
# end the fold in either buffer.
@pytest.mark.parametrize("name,count,steps", [
    ("r10_8_1", 1, 2), ("r10_8_1", 2, 3), ("r10_8_1", 3, 1), ("r10_8_1", 5, 2), ("r10_8_1", 9, 1), ("r10_8_1", 17, 3),
    ("r10_6_4", 1, 3), ("r10_6_4", 16, 2), ("r11_3_1", 1, 1), ("r11_7_3", 2, 3), ("r11_7_3", 16, 1), ("r12_5_2", 3, 2),
    ("r12_4_1", 1, 2), ("r13_3_1", 1, 3), ("r13_5_4", 4, 2)])
def test_fold_parity(name, count, steps):
    p = pair(name, wid=60)
    g = np.random.default_rng(count)
    keys = p.keys([3 << k for k in range(steps)])
    both = [p.encrypt_both(ckks.encode(g.uniform(-1, 1, p.par.slots), p.n, 40), tag=j) for j in range(count)]
    cts = p.ctx.new_ct(count, log_scale=40)
    for j, (dev, _) in enumerate(both):
        cts.t[j * p.ctx.ct_words:(j + 1) * p.ctx.ct_words] = dev.t
    say(f"[fold] {name} {count} ciphertexts, {steps} steps")
    p.ctx.rotate_sum(cts, None, 3, steps)
    got = p.export_ct(cts, count)
    for j, (_, orc) in enumerate(both):
        assert np.array_equal(got[j], p.orc.rotate_sum(orc, 3, steps, keys)), j


# 511 giant steps (two launches of the giant sums); one to nine blocks (quartered and plain finishes)
@pytest.mark.parametrize("name,d,B,blocks", [("r10_2_1", 512, 1, 1), ("r10_8_1", 16, 4, 9), ("r11_7_3", 32, 8, 1),
                                             ("r12_4_1", 16, 8, 17), ("r13_5_4", 16, 2, 2)])
def test_diagonal_product_parity(name, d, B, blocks):
    p = pair(name, wid=61)
    g = np.random.default_rng(d + blocks)
    keys = p.keys(ckks.steps_for_bsgs(d, B))
    ct_dev, ct_orc = p.encrypt_both(ckks.encode(g.uniform(-1, 1, p.par.slots), p.n, 40))
    coeffs = g.integers(-2 ** 30, 2 ** 30, (blocks, d, p.n))
    say(f"[diag] {name} d={d} B={B} blocks={blocks}")
    bufs = [p.ctx.encode_db_block_int(c) for c in coeffs]
    got = p.export_ct(p.ctx.score_block(ct_dev, bufs, d, 1, B), blocks)
    rots = p.orc.baby_rotations(ct_orc, B, keys)
    for j in {0, blocks - 1}:
        pts = np.stack([ckks.to_residues(c, p.par.q) for c in coeffs[j]]).reshape(d // B, B, p.par.L, p.n)
        assert np.array_equal(got[j], p.orc.bsgs_block(rots, pts, B, d // B, keys)), j
