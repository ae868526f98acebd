"""GPU parity of the FP64-word kernel's 32 x 32 tiles against the exact oracle
(tolerance 0): two register slots of loads in flight, and one or two groups of
waves sharing a workgroup's k-range, at the edges of stages, groups and tails.
"""
import sys

import numpy as np
import pytest

import mmp_inputs as gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mmp = pytest.importorskip("paper_2601_07508_amd")

P52, P50, P44, P36, P25 = 4503599627370449, 1125899906842597, 17592186044399, 68719476731, 33554393


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def run(p, u, v, m, n, k, pad=0, **opts):
    plan = mmp.plan(p, m, n, k, u, v, form=1, tile=3, **opts)
    assert (plan["bm"], plan["bn"]) == (32, 32)
    A = gen.random_matrix(m + k, 1, m, k, p)
    B = gen.random_matrix(n + k, 2, k, n, p)
    A[0, :] = B[:, 0] = p - 1
    print("small tiles", p, u, v, m, n, k, pad, opts, plan["kblock"], plan["slots"], file=sys.stderr, flush=True)
    # entries past a row's end are NaN: a k tail that is not cleared would show
    dA = torch.full((m, k + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :k]
    dB = torch.full((k, n + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :n]
    dA.copy_(torch.from_numpy(A.astype(np.float64)))
    dB.copy_(torch.from_numpy(B.astype(np.float64)))
    store = torch.full((m + 1, n + pad), -1.0, dtype=torch.float64, device="cuda")
    mmp.mm_modp_async(dA, dB, store[:m, :n], p, u, v, form=1, tile=3, **opts)
    got = store.cpu().numpy()
    want = oracle.mm_modp(p, A, B).astype(np.float64)
    assert np.array_equal(got[:m, :n], want) and not np.signbit(got[:m, :n]).any()
    assert (got[m:] == -1.0).all() and (got[:, n:] == -1.0).all()


# whole stages of 16 k-terms: 1, 2 and 3, both sides of the 8 and 16 from which two
# groups share the range (an odd count leaves the second group a stage of zeros),
# and a tail of one k-term
@pytest.mark.parametrize("k", [1, 16, 17, 33, 48, 113, 128, 129, 240, 255, 256, 257, 272, 273, 1000])
@pytest.mark.parametrize("p,u,v", [(P25, 1, 1), (P36, 1, 3), (P44, 2, 2), (P52, 3, 2)])
def test_stages(p, u, v, k):
    run(p, u, v, 33, 65, k, pad=3)


# padded stages (blocks shorter than their slots), reductions with corrections,
# longer blocks, centered words, k-ranges
@pytest.mark.parametrize("p,u,v,k,opts", [
    (P50, 2, 2, 500, {}), (P50, 2, 2, 226, {"force_kblock": 7}), (P50, 2, 2, 500, {"force_kblock": 3}),
    (P50, 2, 2, 1000, {"force_kblock": 5}), (P25, 1, 1, 700, {"force_kblock": 4}), (P44, 2, 2, 500, {"strict_fmod": True}),
    (P50, 2, 2, 611, {"extended_block": True}), (P50, 2, 2, 611, {"centered_words": True}),
    (P52, 2, 4, 700, {"centered_words": True}), (P44, 2, 2, 2100, {"splits": 3}), (P36, 1, 3, 5000, {"splits": 7}),
    (P25, 1, 1, 300, {"splits": 16}),
])
def test_classes(p, u, v, k, opts):
    run(p, u, v, 40, 95, k, **opts)


# 256 workgroups (two groups of waves) and one row of tiles more (one group)
@pytest.mark.parametrize("m", [512, 513])
def test_workgroups(m):
    run(P44, 2, 2, m, 512, 300)


def test_batch_of_unequal_lengths():
    # one launch: the shortest product decides on the groups
    for ks in ((300, 700, 256), (300, 20, 700)):
        jobs, wants = [], []
        for i, k in enumerate(ks):
            A = gen.random_matrix(i, 3, 40 + i, k, P44)
            B = gen.random_matrix(i, 4, k, 70 - i, P44)
            dA, dB = (torch.from_numpy(x.astype(np.float64)).cuda() for x in (A, B))
            jobs.append((dA, dB, torch.full((40 + i, 70 - i), -1.0, dtype=torch.float64, device="cuda"), P44, 2, 2))
            wants.append(oracle.mm_modp(P44, A, B).astype(np.float64))
        mmp.mm_modp_batched(jobs)
        for j, w in zip(jobs, wants):
            assert np.array_equal(j[2].cpu().numpy(), w)
