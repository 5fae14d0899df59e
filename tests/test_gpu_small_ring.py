"""GPU parity of the fused key switch and rescale at N = 4096: digits of one to
three primes, a last digit of one prime, seed-expanded and stored keys in one
batch, product sources, batches on both sides of the sizes at which the general
pipeline takes over, rescales of several ciphertexts, in place and over the last
limb that they read.  Bit-exact against the oracle on uniform residues."""
import numpy as np
import pytest
import torch

import synth
from oracle import ckks as C
from tests.gpu_helpers import first_mismatch, need_gpu, step, to_dev, to_host

pytestmark = pytest.mark.gpu
SEED = 23


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _residues(P, level, i):
    return np.stack([synth.uniform_residues(SEED, f"c{t}", P.qs(level), P.n, i)
                     for t in range(2)], axis=1)


def _eq(dev, want, what):
    got = to_host(dev).reshape(want.shape)
    assert np.array_equal(got, want), f"{what}: {first_mismatch(got, want)}"


# the limits: 14 | 15 sources of 8 x 9 extended rows in the ModUp, 5 | 6 jobs of 29
# rows in the ModDown (alpha 3); up to 15 digits in groups of three for the
# seed-expanded half; alpha 4 takes the general pipeline
@pytest.mark.parametrize("bits,L,alpha,level,count", [
    (50, 3, 1, 3, 1), (36, 3, 1, 2, 5), (50, 8, 1, 8, 14), (50, 8, 1, 8, 15), (45, 7, 2, 7, 1),
    (50, 7, 3, 7, 2), (50, 6, 3, 5, 32), (50, 16, 1, 15, 3), (36, 29, 3, 29, 5),
    (36, 29, 3, 29, 6), (50, 5, 4, 5, 2),
])
def test_small_ring(bits, L, alpha, level, count):
    from paper_2608_17442_amd import fesc as F
    P = C.params_small(12, bits, L, alpha)
    ctx = F.Context(P.log_n, P.q, P.p)
    s = synth.secret(SEED, P.n)
    sk, s_dev = C.secret_key(P, s), torch.from_numpy(s).cuda()
    steps = [3, -5]
    g_seed, keys = P.galois_elt(-5), {}
    step(f"keys L={L} alpha={alpha}")
    w, e = synth.switch_key_seed_draws(SEED, P.ext(P.L), P.n, P.dnum, g_seed)
    ctx.keygen_seeded(g_seed, s_dev, w, torch.from_numpy(e).cuda())
    keys[g_seed] = C.keygen_seeded(P, sk, w, e, g_seed)
    for g in (0, P.galois_elt(3)):
        mods = P.ext(P.L)
        keys[g] = np.stack([np.stack([synth.uniform_residues(SEED, f"k{g}{t}", mods, P.n, j)
                                      for t in range(2)], axis=1) for j in range(P.dnum)])
        ctx.key_load(g, to_dev(keys[g]))
    kinds = min(count, 3)
    cts = [_residues(P, level, i) for i in range(kinds)]
    host = [cts[i % kinds] for i in range(count)]
    dev = [to_dev(c).reshape(-1) for c in host]
    pick = sorted({0, count // 2, count - 1})
    r = [steps[i % 2] for i in range(count)]

    def fresh(rows):
        return [torch.zeros(rows * 2 * P.n, dtype=torch.int64, device="cuda") for _ in dev]

    step(f"rotate count={count} level={level}")
    outs = fresh(level)
    ctx.rotate_batch(dev, r, outs, level)
    for i in pick:
        _eq(outs[i], C.rotate(P, host[i], r[i], keys), f"rotate {i}")
    step("hoisted")
    hoisted = [torch.zeros_like(dev[0]) for _ in steps]
    ctx.rotate_hoisted(dev[0], steps, hoisted, level)
    for o, want in zip(hoisted, C.rotate_hoisted(P, host[0], steps, keys)):
        _eq(o, want, "hoisted")
    step("products")
    outs = fresh(level - 1)
    ctx.mul_relin_rescale(dev, dev[::-1], outs, level)
    for i in pick:
        _eq(outs[i], C.mul_relin_rescale(P, host[i], host[count - 1 - i], keys[0]), f"merged {i}")
    prod = torch.zeros_like(dev[0])
    ctx.mul_relin(dev[0], dev[-1], prod, level)
    _eq(prod, C.mul_relin(P, host[0], host[-1], keys[0]), "product")
    step("rescale")
    low = torch.zeros((level - 1) * 2 * P.n, dtype=torch.int64, device="cuda")
    ctx.rescale(dev[0], low, level)
    _eq(low, C.rescale(P, host[0]), "rescale")
    step("in place: a square, a rotation, a rescale")
    ctx.mul_relin(prod, prod, prod, level)
    _eq(prod, C.mul_relin(P, *2 * [C.mul_relin(P, host[0], host[-1], keys[0])], keys[0]), "square")
    ctx.rotate(dev[0], dev[0], level, r[0])
    _eq(dev[0], C.rotate(P, host[0], r[0], keys), "rotation in place")
    ctx.rescale(dev[0], dev[0], level)
    want = C.rescale(P, C.rotate(P, host[0], r[0], keys))
    _eq(dev[0][:want.size], want, "rescale in place")


# 16 ciphertexts per launch: 16 x 32 rows are the limit of the fused rescale, a
# rest of one takes it on either side
@pytest.mark.parametrize("level,n_out", [(2, 3), (33, 17), (34, 16), (34, 17)])
def test_rescale_of_several(level, n_out):
    """The rescale of a matrix-vector product's outputs (one term each)."""
    from paper_2608_17442_amd import fesc as F
    P = C.params_small(12, 36, level, 3)
    ctx = F.Context(P.log_n, P.q, P.p)
    x = _residues(P, level, 0)
    pool = [synth.uniform_residues(SEED, "d", P.qs(level), P.n, i) for i in range(3)]
    dev = [to_dev(p).reshape(-1) for p in pool]
    plan = F.MatvecPlan(ctx, level, 1, n_out, 1, 1, 1, False, True,
                        diags=[dev[b % 3] for b in range(n_out)])
    outs = [torch.zeros((level - 1) * 2 * P.n, dtype=torch.int64, device="cuda")
            for _ in range(n_out)]
    step(f"rescale of {n_out} outputs, level {level}")
    plan([to_dev(x).reshape(-1)], outs)
    want = [C.rescale(P, C.mul_plain(P, x, p)) for p in pool]
    for b, o in enumerate(outs):
        _eq(o, want[b % 3], f"output {b}")


@pytest.mark.parametrize("log_n", [12, 13])
def test_rescale_over_its_last_limb(log_n):
    """An output that starts at the last limb of the input: every row reads that
    limb, so the rows cannot be one launch."""
    from paper_2608_17442_amd import fesc as F
    level = 5
    P = C.params_small(log_n, 50, level, 1)
    ctx = F.Context(P.log_n, P.q, P.p)
    x, limb = _residues(P, level, 0), 2 * P.n
    buf = torch.zeros((2 * level - 2) * limb, dtype=torch.int64, device="cuda")
    buf[:level * limb] = to_dev(x).reshape(-1)
    step(f"rescale over the last limb, N=2^{log_n}")
    ctx.rescale(buf[:level * limb], buf[(level - 1) * limb:], level)
    _eq(buf[(level - 1) * limb:], C.rescale(P, x), "over the last limb")
    _eq(buf[:(level - 1) * limb], x[:-1], "the other limbs")
