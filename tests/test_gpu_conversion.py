"""GPU parity of the key switch's basis conversions over ring degrees, digit
sizes and batch sizes: the matrix-core products (digits of four to eight
primes, with ninth source in the merged product), the VALU conversion (shorter
digits and those past eight), digits finished by the conversion and by a pass of
their own, quads of targets dealt over workgroups and partial last quads.
Bit-exact against the oracle on uniform residues."""
import numpy as np
import pytest
import torch

import synth
from oracle import ckks as C
from tests.gpu_helpers import first_mismatch, need_gpu, step, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _residues(P, level, tag, i):
    return np.stack([synth.uniform_residues(21, f"{tag}{t}", P.qs(level), P.n, i)
                     for t in range(2)], axis=1)


def _key(P, seed):
    mods = P.ext(P.L)
    return np.stack([np.stack([synth.uniform_residues(seed, f"k{t}", mods, P.n, j)
                               for t in range(2)], axis=1) for j in range(P.dnum)])


# alpha 3 | 4: the two sides of the choice of unit; 8: nine sources in the
# merged product; 9: past the matrix-core tables; levels with a last digit of
# one prime or a single one shorter than alpha, and target counts of every
# remainder mod 4; digits past the tables in each of the VALU's forms (13, 9 and, a
# batch with few rows, 14, 9: fused, 16, 12: one target per workgroup, 14, 12: three).
# alpha 8 at every ring on both sides of 8 M digits = 768, past which the matrix cores
# read digits that a pass of their own has finished (no such pass at N = 4096)
@pytest.mark.parametrize("log_n,bits,L,alpha,level,count", [
    (12, 50, 7, 3, 7, 1), (12, 50, 9, 4, 9, 1), (12, 36, 10, 4, 10, 33),
    (13, 50, 9, 8, 9, 1), (13, 36, 6, 5, 6, 5), (14, 50, 9, 8, 9, 2), (14, 45, 10, 9, 10, 1),
    (15, 50, 7, 6, 7, 1), (15, 50, 4, 3, 4, 24), (16, 50, 5, 4, 5, 1), (16, 36, 3, 2, 3, 1),
    (16, 50, 5, 12, 5, 1), (13, 45, 9, 9, 9, 1), (14, 36, 12, 12, 12, 8),
    (15, 50, 3, 3, 3, 24), (14, 50, 4, 9, 4, 16),
    (12, 50, 9, 8, 9, 2), (13, 50, 9, 8, 9, 32), (14, 50, 9, 8, 9, 16), (15, 50, 9, 8, 9, 1),
    (15, 50, 9, 8, 9, 8), (16, 50, 9, 8, 9, 1), (16, 50, 9, 8, 9, 4),
])
def test_key_switch_conversions(log_n, bits, L, alpha, level, count):
    from paper_2608_17442_amd import fesc as F
    P = C.params_small(log_n, bits, L, alpha)
    ctx = F.Context(P.log_n, P.q, P.p)
    r = 3
    keys = {P.galois_elt(r): _key(P, 31), 0: _key(P, 32)}
    for g, k in keys.items():
        ctx.key_load(g, to_dev(k))
    cts = [_residues(P, level, "c", i % 3) for i in range(count)]
    dev = [to_dev(c).reshape(-1) for c in cts]
    outs = [torch.zeros_like(d) for d in dev]
    step(f"rotate log_n={log_n} alpha={alpha} level={level} count={count}")
    ctx.rotate_batch(dev, [r] * count, outs, level)
    want = [C.rotate(P, c, r, keys) for c in cts[:3]]
    for i, o in enumerate(outs):
        got = to_host(o).reshape(want[i % 3].shape)
        assert np.array_equal(got, want[i % 3]), first_mismatch(got, want[i % 3])
    step("merged product")
    outs = [torch.zeros((level - 1) * 2 * P.n, dtype=torch.int64, device="cuda") for _ in dev]
    ctx.mul_relin_rescale(dev, dev[::-1], outs, level)
    for i in {0, count // 2, count - 1}:
        want = C.mul_relin_rescale(P, cts[i], cts[count - 1 - i], keys[0])
        got = to_host(outs[i]).reshape(want.shape)
        assert np.array_equal(got, want), first_mismatch(got, want)
