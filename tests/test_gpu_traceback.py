"""The segmented traceback of the rotating survivor layouts against the
oracle: emitted ranges that do not start on a word, odd stage counts, frames
around the 32-stage blocks and segment edges, several frames per wavefront,
segments of one and of several blocks, ties everywhere (segments that must be
traced again)."""
import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import Code, CODE_K5, CODE_K7, CODE_K9

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CODES = [Code.from_octal(3, ["7", "5"]), Code.from_octal(4, ["15", "17"]), CODE_K5,
         Code.from_octal(6, ["53", "75"]), CODE_K7, Code.from_octal(8, ["247", "371"]), CODE_K9]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _check(code, lens, begins, dtype, radix, seed, ties):
    rng = np.random.default_rng(seed)
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    ofr = np.zeros(len(lens), oracle.FRAME_DTYPE)
    off = boff = 0
    for k, (S, ob) in enumerate(zip(lens, begins)):
        ob = min(ob, S)
        n = max(0, S - ob - int(rng.integers(0, 4)))
        known, zero = int(rng.integers(0, 2)), int(rng.integers(0, 2))
        fr[k] = (off, boff, S, ob, n, 0, known | 2 * zero)
        ofr[k] = (off, boff, S, ob, n, known, 0 if zero else -1, 0)
        off += S * code.beta
        boff += (n + 31) // 32 * 32
    if ties:
        llr = rng.integers(-1, 2, off)
    else:
        # a noisy all-zero codeword
        llr = np.clip(np.rint(rng.normal(20, 14, off)), -127, 127)
    llr = llr.astype({"i8": np.int8, "f32": np.float32}[dtype])
    print("traceback", code.K, dtype, radix, len(lens), ties, flush=True)
    plan = mv.Plan([code], fr, dtype, radix)
    w, _, _ = plan.decode(torch.from_numpy(llr).to("cuda:0"))
    got = mv.unpack_bits(w.cpu().numpy(), boff)
    ob, _, _, _ = oracle.decode_frames([code], ofr, llr, oracle.I64 if dtype == "i8" else oracle.F32,
                                       boff)
    for k in range(len(fr)):
        a, n = int(fr[k]["bit_offset"]), int(fr[k]["n_out"])
        np.testing.assert_array_equal(got[a:a + n], ob[a:a + n])
        assert not got[a + n:a + (n + 31) // 32 * 32].any()  # the last word is zero-padded


@pytest.mark.parametrize("code", CODES, ids=lambda c: "K%d" % c.K)
@pytest.mark.parametrize("dtype,radix", [("f32", 2), ("i8", 4)])
def test_edges(code, dtype, radix):
    if radix == 4 and code.K not in (5, 7):
        radix = 2
    lens = [1, 2, 3, 7, 31, 32, 33, 34, 63, 64, 65, 95, 96, 97, 127, 129, 255, 257, 1023, 1055, 2047,
            2081, 2082]
    for ties in (False, True):
        for shift in (0, 1, 17, 31, 32, 47):
            _check(code, lens, [shift + (k % 3) for k in range(len(lens))], dtype, radix,
                   100 * code.K + shift, ties)


@pytest.mark.parametrize("code,dtype", [(CODE_K5, "i8"), (CODE_K7, "i8"), (CODE_K7, "f32"),
                                        (CODE_K9, "i8")],
                         ids=["k5-i8", "k7-i8", "k7-f32", "k9-i8"])
def test_long_segments(code, dtype):
    """Enough stages that a lane traces several blocks."""
    F = 9000 if code.K < 9 else 4000
    lens = [1111 + 2 * (k % 40) + (k % 7 == 0) for k in range(F)]
    _check(code, lens, [(k // 40) % 3 * 33 for k in range(F)], dtype,
           4 if dtype == "i8" and code.K < 9 else 2, 77, False)
