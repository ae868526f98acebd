"""Which kernels a call runs on, where the plan alone does not say (the launch phases do)."""
import sys

import numpy as np
import pytest

import mmp_inputs as gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mmp = pytest.importorskip("paper_2601_07508_amd")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def timed(call):
    """The launch phases of one call."""
    mmp.timers_read(reset=True)
    mmp.timers_enable(True)
    call()
    torch.cuda.synchronize()
    mmp.timers_enable(False)
    return mmp.timers_read(reset=True)


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def test_strict_reductions_keep_fp64_words():
    # planned on FP64 words, estimated faster on INT8 words: an option that asks for
    # the words' complete reductions is not passed over
    p, m, n, k = 1125899906842597, 300, 333, 800
    assert mmp.plan(p, m, n, k, strict_fmod=True)["form"] == mmp.FORM_FP64_WORDS
    A, B = gen.random_matrix(1, 1, m, k, p), gen.random_matrix(1, 2, k, n, p)
    dA, dB, C = dev(A), dev(B), torch.empty((m, n), dtype=torch.float64, device="cuda")
    want = oracle.mm_modp(p, A, B).astype(np.float64)
    for strict in (False, True):
        C.fill_(-1.0)
        say("strict", strict)
        phases = timed(lambda: mmp.mm_modp_async(dA, dB, C, p, strict_fmod=strict))
        assert ("fp64_words" in phases) == strict, phases
        assert np.array_equal(C.cpu().numpy(), want)
