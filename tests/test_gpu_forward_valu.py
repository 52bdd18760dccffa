"""The radix-2 forward of K <= 7 with exchanges in the vector ALU against the
oracle: stage counts around its 32-stage blocks and its periods, wavefronts
whose last frame group is incomplete, all rates and types; and soft values
that its short form does not take (huge, infinite, NaN)."""
import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import Code, CODE_K5, CODE_K7

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CODES = [Code.from_octal(3, ["7", "5"]), Code.from_octal(4, ["15", "17", "13"]), CODE_K5,
         Code.from_octal(5, ["37", "33", "25", "35"]), Code.from_octal(6, ["53", "75"]), CODE_K7,
         Code.from_octal(7, ["133", "171", "145"])]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _frames(code, lens, flags):
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    ofr = np.zeros(len(lens), oracle.FRAME_DTYPE)
    off = boff = 0
    for k, (S, fl) in enumerate(zip(lens, flags)):
        fr[k] = (off, boff, S, 0, S, 0, fl)
        ofr[k] = (off, boff, S, 0, S, fl & 1, 0 if fl & 2 else -1, 0)
        off += S * code.beta
        boff += (S + 31) // 32 * 32
    return fr, ofr, off, boff


def _check(code, fr, ofr, llr, boff, dtype, skip=()):
    plan = mv.Plan([code], fr, dtype, 2)
    w, m, e = plan.decode(torch.from_numpy(llr).to("cuda:0"))
    got, m, e = mv.unpack_bits(w.cpu().numpy(), boff), m.cpu().numpy(), e.cpu().numpy()
    ref = llr.astype(np.float32) if dtype == "f16" else llr
    ob, om, oe, _ = oracle.decode_frames([code], ofr, ref,
                                         oracle.I64 if dtype == "i8" else oracle.F32, boff)
    for k in range(len(fr)):
        if k in skip:
            continue
        a, n = int(fr[k]["bit_offset"]), int(fr[k]["n_out"])
        np.testing.assert_array_equal(got[a:a + n], ob[a:a + n])
        assert e[k] == oe[k] and m[k] == om[k]


@pytest.mark.parametrize("code", CODES, ids=lambda c: "K%d_%d" % (c.K, c.beta))
@pytest.mark.parametrize("dtype", ["f32", "f16", "i8"])
def test_blocks_and_periods(code, dtype):
    n = code.K - 1
    period = 32 * n // np.gcd(32, n)
    lens = sorted({1, 2, n, 31, 32, 33, 63, 64, 65, period - 1, period, period + 1, 2 * period - 31,
                   3 * period + 32, 3 * period + 63, 5 * period}) * 3
    rng = np.random.default_rng(31 * code.K + code.beta)
    fr, ofr, total, boff = _frames(code, lens, rng.integers(0, 4, len(lens)))
    for x in (rng.normal(1, 2, total) * 8, np.rint(rng.normal(0, 1, total)), np.zeros(total)):
        x = np.clip(np.rint(x), -128, 127) if dtype == "i8" else x
        x = x.astype({"f32": np.float32, "f16": np.float16, "i8": np.int8}[dtype])
        print("valu", code.K, code.beta, dtype, flush=True)
        _check(code, fr, ofr, x, boff, dtype)


@pytest.mark.parametrize("code", [CODE_K5, CODE_K7], ids=["K5", "K7"])
def test_huge_and_infinite_soft_values(code):
    rng = np.random.default_rng(9)
    lens = [40, 97, 150, 97, 300, 97, 700, 700]
    fr, ofr, total, boff = _frames(code, lens, [1, 0, 3, 2, 1, 3, 0, 1])
    x = rng.normal(1, 2, total).astype(np.float32)
    huge = rng.random(total) < 0.01
    x[huge] *= np.float32(1e35)  # sums stay finite
    print("huge", code.K, flush=True)
    _check(code, fr, ofr, x, boff, "f32")
    # one infinity a frame, after every state can be reached: all metrics
    # become +inf there and every later decision is a tie
    for k, S in enumerate(lens):
        t = int(rng.integers(code.K, S))
        x[int(fr[k]["llr_offset"]) + t * code.beta] = np.inf if k % 2 else -np.inf
    print("infinite", code.K, flush=True)
    _check(code, fr, ofr, x, boff, "f32")


def test_nan_stays_in_its_frame():
    """Frames that share a wavefront with one holding NaNs are unaffected."""
    rng = np.random.default_rng(10)
    lens = [500] * 8  # K = 5: four frames per wavefront
    fr, ofr, total, boff = _frames(CODE_K5, lens, [3] * 8)
    x = rng.normal(1, 2, total).astype(np.float32)
    x[int(fr[2]["llr_offset"]) + 333] = np.nan
    x[int(fr[5]["llr_offset"]) + 1] = np.nan
    print("nan", flush=True)
    _check(CODE_K5, fr, ofr, x, boff, "f32", skip=(2, 5))
