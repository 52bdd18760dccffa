"""The packed int8 forward of K = 8 and 9 (two states per register, radix-4
digits collected in the metrics) against the oracle: stage counts around its
groups, table blocks and trips, odd counts, mixed starts and ends, soft values
that drive the 16-bit metrics to the edges of their range, and frames split in
time whose boundaries have to be repaired."""
import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import Code, encode_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CODES = [Code.from_octal(8, ["247", "371"]), Code.from_octal(8, ["225", "331", "367"]),
         Code.from_octal(9, ["561", "753"]), Code.from_octal(9, ["557", "663", "711"]),
         # outputs that are all alike: the largest spread of the metrics
         Code.from_octal(9, ["401", "401", "401"]), Code.from_octal(8, ["201", "201"])]
IDS = ["K%d-%s" % (c.K, "_".join("%o" % g for g in c.gens)) for c in CODES]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _check(code, lens, flags, llr_of, split=True, out_of=None):
    beta = len(code.gens)
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    ofr = np.zeros(len(lens), oracle.FRAME_DTYPE)
    off, boff, parts = 1, 0, []  # soft values at odd addresses
    for k, (S, fl) in enumerate(zip(lens, flags)):
        ob, n = out_of(k, S) if out_of else (0, S)
        fr[k] = (off, boff, S, ob, n, 0, fl)
        ofr[k] = (off, boff, S, ob, n, fl & 1, 0 if fl & 2 else -1, 0)
        parts.append(llr_of(k, S))
        off += beta * S
        boff += (n + 31) // 32 * 32
    x = np.concatenate([np.zeros(1)] + parts).astype(np.int8)
    print("packed", code.K, [oct(g) for g in code.gens], len(lens), split, flush=True)
    plan = mv.Plan([code], fr, "i8", 2, split=split)
    assert "two states per register" in plan.describe()
    w, m, e = plan.decode(torch.from_numpy(x).to("cuda:0"))
    ob, om, oe, _ = oracle.decode_frames([code], ofr, x, oracle.I64, boff)
    np.testing.assert_array_equal(m.cpu().numpy(), om)
    np.testing.assert_array_equal(e.cpu().numpy(), oe)
    got = mv.unpack_bits(w.cpu().numpy(), boff)
    for k in range(len(fr)):
        a, n = int(fr[k]["bit_offset"]), int(fr[k]["n_out"])
        np.testing.assert_array_equal(got[a:a + n], ob[a:a + n])


LENS = [1, 2, 3, 6, 7, 8, 9, 15, 16, 17, 27, 28, 29, 31, 32, 33, 55, 56, 57, 62, 63, 64, 65, 66, 110,
        111, 112, 113, 114, 127, 128, 129, 223, 225, 257]


@pytest.mark.parametrize("code", CODES, ids=IDS)
def test_blocks_and_trips(code):
    rng = np.random.default_rng(11 * code.K + len(code.gens))
    flags = rng.integers(0, 4, len(LENS))
    beta = len(code.gens)
    _check(code, LENS, flags, lambda k, S: rng.integers(-128, 128, beta * S))
    _check(code, LENS, flags, lambda k, S: rng.integers(-1, 2, beta * S),
           out_of=lambda k, S: (k % 5 * S // 5, S - k % 5 * S // 5 - k % 2 * (S // 7)))


@pytest.mark.parametrize("code", CODES, ids=IDS)
def test_range_edges(code):
    rng = np.random.default_rng(13 * code.K + len(code.gens))
    beta, S = len(code.gens), 700

    def word(k, S):
        bits = [np.ones(S), rng.integers(0, 2, S), np.arange(S) // 9 % 2, np.zeros(S),
                (rng.random(S) < 0.9)][k % 5].astype(np.uint8)
        c = encode_bits(code, bits[None], False)[0].reshape(-1)
        x = np.where(c == 1, -128, 127) if k % 2 else np.where(c == 1, 127, -128)
        if k >= 10:  # bursts of another codeword
            d = encode_bits(code, rng.integers(0, 2, S).astype(np.uint8)[None], False)[0].reshape(-1)
            x = np.where(np.arange(beta * S) // 64 % 3 == 0, np.where(d == 1, -128, 127), x)
        return x

    _check(code, [S + k % 2 for k in range(24)], rng.integers(0, 4, 24), word)
    _check(code, [300, 301, 302, 303], [0, 1, 2, 3],
           lambda k, n: np.full(beta * n, [-128, 127, -127, 126][k]))


@pytest.mark.parametrize("code", CODES[:4], ids=IDS[:4])
def test_split_and_whole_agree_on_noise(code):
    """Frames long enough to be split in time, pure noise: boundaries that
    disagree are repaired."""
    rng = np.random.default_rng(17 * code.K)
    beta = len(code.gens)
    lens = [5001, 5000, 2049, 2048, 9003]
    x = [rng.integers(-128, 128, beta * S) if k % 2 else
         np.rint(rng.normal(0, 1, beta * S)).clip(-128, 127) for k, S in enumerate(lens)]
    x[4][:] = 0  # ties only
    for split in (True, False):
        _check(code, lens, [0, 1, 2, 3, 1], lambda k, S: x[k], split)


@pytest.mark.parametrize("code", CODES[4:], ids=IDS[4:])
@pytest.mark.parametrize("S", [4096, 6001])
def test_boundaries_that_never_merge(code, S):
    """Chains of two states keep the metric difference they start with under
    soft values of constant size: no warm-up finds it, every boundary is
    repaired."""
    rng = np.random.default_rng(S)
    beta = len(code.gens)
    x = [np.full(beta * S, 100), np.repeat(rng.choice([-90, 90], S), beta),
         np.repeat(rng.choice([-128, 127], S), beta)]
    _check(code, [S] * 3, [1, 3, 1], lambda k, n: x[k])
