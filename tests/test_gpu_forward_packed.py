"""The packed int8 forward of K = 5 and 7 (two frames per register, decisions
collected in the metrics) against the oracle: stage counts around its blocks
and trips, odd frame counts, mixed starts and ends, soft values that drive the
16-bit metrics to the edges of their range, and codes on both sides of the
spread that sets its range-control interval."""
import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import Code, CODE_K5, CODE_K7, encode_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (101, 101): six stages can differ in all twelve outputs, the most there is
CODE_K7_WIDE = Code.from_octal(7, ["101", "101"])
CODE_K7_B = Code.from_octal(7, ["117", "155"])


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _check(code, lens, flags, llr_of, variant, split=True):
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    ofr = np.zeros(len(lens), oracle.FRAME_DTYPE)
    off, boff, parts = 1, 0, []  # soft values at odd addresses
    for k, (S, fl) in enumerate(zip(lens, flags)):
        fr[k] = (off, boff, S, 0, S, 0, fl)
        ofr[k] = (off, boff, S, 0, S, fl & 1, 0 if fl & 2 else -1, 0)
        parts.append(llr_of(k, S))
        off += 2 * S
        boff += (S + 31) // 32 * 32
    x = np.concatenate([np.zeros(1)] + parts).astype(np.int8)
    print("packed", code.K, [oct(g) for g in code.gens], variant, len(lens), split, flush=True)
    plan = mv.Plan([code], fr, "i8", 4, variant=variant, split=split)
    assert "packed" in plan.describe()
    w, m, e = plan.decode(torch.from_numpy(x).to("cuda:0"))
    ob, om, oe, _ = oracle.decode_frames([code], ofr, x, oracle.I64, boff)
    np.testing.assert_array_equal(m.cpu().numpy(), om)
    np.testing.assert_array_equal(e.cpu().numpy(), oe)
    got = mv.unpack_bits(w.cpu().numpy(), boff)
    for k in range(len(fr)):
        a, n = int(fr[k]["bit_offset"]), int(fr[k]["n_out"])
        np.testing.assert_array_equal(got[a:a + n], ob[a:a + n])


CASES = [(CODE_K5, 0), (CODE_K7, 4), (CODE_K7, 5), (CODE_K7_B, 5), (CODE_K7_WIDE, 4),
         (CODE_K7_WIDE, 5)]
IDS = ["%s-v%d" % ("_".join("%o" % g for g in c.gens), v) for c, v in CASES]


@pytest.mark.parametrize("code,variant", CASES, ids=IDS)
def test_blocks_and_trips(code, variant):
    rng = np.random.default_rng(5 * code.K + variant)
    lens = [1, 2, 3, 5, 6, 7, 8, 15, 16, 17, 18, 31, 33, 47, 48, 49, 50, 94, 95, 96, 97, 98, 143, 144,
            191, 193, 200, 289]
    lens = [s for s in lens for _ in range(3)]  # pairs, and a frame alone
    flags = rng.integers(0, 4, len(lens))
    _check(code, lens, flags, lambda k, S: rng.integers(-128, 128, 2 * S), variant)
    _check(code, lens, flags, lambda k, S: rng.integers(-1, 2, 2 * S), variant)


@pytest.mark.parametrize("code,variant", CASES, ids=IDS)
def test_range_edges(code, variant):
    """Saturated codewords: the best metric grows by up to 256 a stage, the
    spread is the largest the code allows; and the same with the sign turned,
    constant and alternating values."""
    rng = np.random.default_rng(50 * code.K + variant)
    S = 1500

    def word(k, S):
        bits = [np.ones(S), rng.integers(0, 2, S), np.arange(S) // 7 % 2, np.zeros(S),
                (rng.random(S) < 0.9)][k % 5].astype(np.uint8)
        c = encode_bits(code, bits[None], False)[0].reshape(-1)
        x = np.where(c == 1, -128, 127) if k % 2 else np.where(c == 1, 127, -128)
        if k >= 10:  # bursts of another codeword
            d = encode_bits(code, rng.integers(0, 2, S).astype(np.uint8)[None], False)[0].reshape(-1)
            x = np.where(np.arange(2 * S) // 64 % 3 == 0, np.where(d == 1, -128, 127), x)
        return x

    consts = [-128, 127]
    flags = rng.integers(0, 4, 24)
    _check(code, [S + k % 2 for k in range(24)], flags, lambda k, n: word(k, n), variant)
    _check(code, [300] * 6, [0, 1, 2, 3, 0, 1],
           lambda k, n: np.full(2 * n, consts[k % 2]) * np.where(np.arange(2 * n) % (k + 1), 1, -1)
           .clip(-1, 1) if k > 1 else np.full(2 * n, consts[k % 2]), variant)


@pytest.mark.parametrize("code,variant", [(CODE_K5, 0), (CODE_K7, 4), (CODE_K7, 5)],
                         ids=["k5", "k7-v4", "k7-v5"])
def test_split_and_whole_agree_on_noise(code, variant):
    """Pure noise: boundaries of frames split in time disagree and the check
    repairs them."""
    rng = np.random.default_rng(77)
    x = [rng.integers(-128, 128, 2 * 4001) for _ in range(11)]
    for split in (True, False):
        _check(code, [4001] * 11, [k % 4 for k in range(11)], lambda k, S: x[k], variant, split)


@pytest.mark.parametrize("variant", [4, 5])
def test_boundaries_that_never_merge(variant):
    """Chains of two states keep the metric difference they start with under
    soft values of constant size: no warm-up finds it, every boundary is
    repaired."""
    rng = np.random.default_rng(variant)
    S = 6001
    x = [np.full(2 * S, 100), np.repeat(rng.choice([-90, 90], S), 2),
         np.repeat(rng.choice([-128, 127], S), 2)]
    _check(CODE_K7_WIDE, [S] * 3, [1, 3, 1], lambda k, n: x[k], variant)
