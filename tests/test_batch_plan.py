"""Which products of an AUTO batch leave the FP64 words that their own plan
names for the launches that INT8 words share (host only: the plan shows in the
workspace that the batch asks for)."""
import ctypes

import pytest

pytest.importorskip("torch")  # first, so that the library takes the HIP runtime that torch brings
mmp = pytest.importorskip("paper_2601_07508_amd")

P25, P36, P50 = 33554393, 68719476731, 1125899906842597


def workspace(dims, **opts):
    """mmp_workspace_batched of products (m, n, k, p), or (m, n, k, p, u, v), at addresses that nothing reads."""
    jobs = (mmp.MmpJob * len(dims))()
    at = 1 << 32
    for j, (m, n, k, p, *words) in zip(jobs, dims):
        j.p, j.m, j.n, j.k = p, m, n, k
        j.u, j.v = words or (0, 0)
        j.lda, j.ldb, j.ldc = k, n, n
        j.A, j.B, j.C = at, at + 8 * m * k, at + 8 * (m * k + k * n)
        at += 8 * (m * k + k * n + m * n)
    return mmp.lib().mmp_workspace_batched(jobs, len(dims), ctypes.byref(mmp._opts(**opts)))


def planned_on_fp64(dims):
    return all(mmp.plan(p, m, n, k, splits=1)["form"] == mmp.FORM_FP64_WORDS for m, n, k, p in dims)


# one operand read once bounds them (2 of 16384 x 8 x 32768 at 25 bits: 2.06 ms on
# FP64 words, 4.64 on INT8 words), or a launch or two (2 of 64^3: 17 us against 24),
# or the outputs (2 of 4096 x 4096 x 8 at 25 bits: 69 us against 122)
@pytest.mark.parametrize("dims", [
    [(16384, 8, 32768, P25)] * 2, [(16384, 1, 32768, P36)] * 6, [(4096, 8, 8192, P25)] * 6,
    [(8, 4096, 8192, P25)] * 6, [(64, 64, 64, P36)] * 2, [(128, 128, 128, P50)] * 4, [(512, 512, 64, P25)] * 4,
    [(4096, 4096, 8, P25)] * 6, [(200, 90, 300, P25), (77, 64, 140, P25), (512, 100, 64, P25)],
])
def test_faster_on_fp64_words(dims):
    assert planned_on_fp64(dims)
    assert workspace(dims) == 0


# a launch for each configuration, or long chains with the chip idle
@pytest.mark.parametrize("dims", [
    [(512, 512, 512, P36)] * 4, [(1000, 1, 1000, P50)] * 6, [(16, 16, 65536, P25)] * 2,
    [(2000, 2000, 32, P36)] * 16, [(100 + 9 * i, 400 - 11 * i, 64 + 23 * i, (1 << (20 + 2 * i)) - 1) for i in range(16)],
])
def test_faster_on_int8_words(dims):
    assert planned_on_fp64(dims)
    assert workspace(dims) > 0


def test_joins_others_launches():
    # a product on INT8 words anyway: another one shares its launches
    large, small = (2048, 2048, 2048, P50), (96, 80, 200, P36)
    alone = workspace([large, (0, 0, 0, P36)])
    assert planned_on_fp64([small]) and alone > 0
    assert workspace([small, small]) == 0 and workspace([large, small]) > alone


def test_memory_that_no_plan_calls_for_is_bounded():
    # faster on INT8 words one and all, 2.6 to 5 GB of planes each
    dims = [(16384, 1, 32768, P50)] * 16
    assert planned_on_fp64(dims)
    assert 0 < workspace(dims) <= (8 << 30) + 16 * 256


@pytest.mark.parametrize("option", ["strict_fmod", "extended_block", "centered_words"])
def test_options_of_fp64_words_keep_them(option):
    dims = [(512, 512, 512, P36)] * 4
    assert mmp.plan(P36, 512, 512, 512, splits=1, **{option: True})["form"] == mmp.FORM_FP64_WORDS
    assert workspace(dims) > 0 and workspace(dims, **{option: True}) == 0


@pytest.mark.parametrize("launch", [1, 2])
def test_batch_option_is_refused_elsewhere(launch):
    # before any device work
    lib, o, best, tried = mmp.lib(), mmp._opts(batch_launch=launch), mmp.MmpPlan(), ctypes.c_int(-1)
    assert lib.mmp_autotune(P36, 64, 64, 64, ctypes.byref(o), ctypes.byref(best), ctypes.byref(tried)) == -1
    fake = [ctypes.c_void_p(0x10000000 * (i + 1)) for i in range(3)]
    args = (ctypes.byref(o), P36, 0, 0, 8, 8, 8, fake[0], 8, fake[1], 8, fake[2], 8, None)
    assert lib.mm_modp_async(*args) == -1 and lib.mm_modp_static(*args) == -1
