"""GPU parity of the projection's plaintext multiply-accumulate over output
counts (every group size, partial last groups, groups that straddle the shared
words of the diagonal bank) and term counts (fewer than, equal to and past
what a split over wavefronts takes), with diagonals from a table and from a
bank, in launches small enough to be split and large enough not to be.
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


SPLIT = [(12, 2, n_out, terms)
         for n_out, terms in [(1, 1), (1, 7), (1, 8), (1, 33), (2, 7), (2, 9), (2, 32), (3, 8), (4, 35),
                              (5, 8), (7, 3), (8, 17), (9, 6), (12, 9), (13, 5), (16, 8), (17, 9),
                              (22, 4), (24, 9), (25, 3), (33, 2), (36, 5)]]
WHOLE = [(16, 2, 1, 9), (16, 2, 3, 8), (16, 2, 6, 9), (16, 2, 24, 3), (16, 2, 17, 2)]


@pytest.mark.parametrize("log_n,level,n_out,terms", SPLIT + WHOLE)
def test_multiply_accumulate(log_n, level, n_out, terms):
    from paper_2608_17442_amd import fesc as F
    P = C.params_small(log_n, 50, level, 1)
    ctx = F.Context(P.log_n, P.q, P.p)
    qs = P.qs(level)
    ins = [np.stack([synth.uniform_residues(41, f"x{t}", qs, P.n, u) for t in range(2)], axis=1)
           for u in range(terms)]
    # a few distinct plaintexts, each output starting at another one
    pool = [synth.uniform_residues(42, "d", qs, P.n, i) for i in range(5)]
    pool[3][:] = 0
    pool[4] = np.stack([np.full(P.n, q - 1, dtype=np.uint64) for q in qs])
    diag = [[pool[(3 * b + u) % 5] for u in range(terms)] for b in range(n_out)]
    dev = [to_dev(p).reshape(-1) for p in pool]
    flat = [dev[(3 * b + u) % 5] for b in range(n_out) for u in range(terms)]
    dins = [to_dev(x).reshape(-1) for x in ins]
    args = (level, terms, n_out, 1, 1, 1, False, False)
    desc = F.matvec_desc(*args)
    bank = torch.full((F.matvec_bank_words(ctx, desc),), -1, dtype=torch.int64, device="cuda")
    F.matvec_bank_pack_many(ctx, desc, bank, 0, torch.stack(flat))
    for kind in ("diags", "bank"):
        plan = F.MatvecPlan(ctx, *args, **{kind: flat if kind == "diags" else bank})
        outs = [torch.zeros(level * 2 * P.n, dtype=torch.int64, device="cuda")
                for _ in range(n_out)]
        step(f"{kind} log_n={log_n} n_out={n_out} terms={terms}")
        plan(dins, outs)
        for b in {0, n_out // 2, n_out - 1, min(11, n_out - 1), min(12, n_out - 1)}:
            want = C.mul_plain(P, ins[0], diag[b][0])
            for u in range(1, terms):
                want = C.ct_add(P, want, C.mul_plain(P, ins[u], diag[b][u]))
            got = to_host(outs[b]).reshape(want.shape)
            assert np.array_equal(got, want), f"{kind} {b}: {first_mismatch(got, want)}"
