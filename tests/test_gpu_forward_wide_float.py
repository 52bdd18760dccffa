"""The K = 8, 9 float forward against the oracle: stage counts around its half
blocks, blocks and trips, one, two and four wavefronts per frame, batches on
both sides of the rule that picks them, and soft values its short form does
not take (huge, infinite)."""
import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import Code, CODE_K9

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CODE_K8 = Code.from_octal(8, ["247", "371"])
CODE_K8_3 = Code.from_octal(8, ["225", "331", "367"])
CODE_K9_4 = Code.from_octal(9, ["463", "535", "733", "745"])


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(code, lens, flags, make, dtype="f32", variant=0):
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    ofr = np.zeros(len(lens), oracle.FRAME_DTYPE)
    off = boff = 0
    for k, (S, fl) in enumerate(zip(lens, flags)):
        fr[k] = (off, boff, S, 0, S, 0, fl)
        ofr[k] = (off, boff, S, 0, S, fl & 1, 0 if fl & 2 else -1, 0)
        off += S * code.beta
        boff += (S + 31) // 32 * 32
    x = make(off, fr).astype({"f32": np.float32, "f16": np.float16}[dtype])
    print("wide float", code.K, code.beta, dtype, variant, len(lens), flush=True)
    plan = mv.Plan([code], fr, dtype, 2, variant=variant)
    w, m, e = plan.decode(torch.from_numpy(x).to("cuda:0"))
    ob, om, oe, _ = oracle.decode_frames([code], ofr, x.astype(np.float32), oracle.F32, boff)
    np.testing.assert_array_equal(e.cpu().numpy(), oe)
    np.testing.assert_array_equal(m.cpu().numpy(), om)
    got = mv.unpack_bits(w.cpu().numpy(), boff)
    for k in range(len(fr)):
        a, n = int(fr[k]["bit_offset"]), int(fr[k]["n_out"])
        np.testing.assert_array_equal(got[a:a + n], ob[a:a + n])


@pytest.mark.parametrize("code,variant", [(CODE_K8, 0), (CODE_K8, 6), (CODE_K8_3, 0), (CODE_K9, 0),
                                          (CODE_K9, 6), (CODE_K9, 7), (CODE_K9_4, 0),
                                          (CODE_K9_4, 7)],
                         ids=lambda v: "K%d_%d" % (v.K, v.beta) if hasattr(v, "K") else "v%d" % v)
@pytest.mark.parametrize("many", [False, True], ids=["few", "many"])
def test_blocks_and_trips(code, variant, many):
    trip = 64 if code.K == 9 else 224
    lens = [1, 15, 16, 17, 31, 32, 33, 47, 49, trip - 1, trip, trip + 1, 2 * trip + 16,
            3 * trip - 17, 5 * trip]
    if many:  # one wavefront per frame by the rule of the default
        lens = [trip + k % 70 for k in range(1500)]
    rng = np.random.default_rng(code.K + 10 * code.beta)
    flags = rng.integers(0, 4, len(lens))
    for make in ((lambda n, fr: rng.normal(1, 2, n) * 8),
                 (lambda n, fr: np.rint(rng.normal(0, 1, n)))):
        _run(code, lens, flags, make, "f32", variant)
        if variant == 0:
            _run(code, lens, flags, make, "f16")


@pytest.mark.parametrize("code,variant", [(CODE_K8, 0), (CODE_K9, 6), (CODE_K9, 7)])
def test_huge_and_infinite_soft_values(code, variant):
    rng = np.random.default_rng(19)
    lens = [50, 97, 150, 300, 700, 700]

    def huge(n, fr):
        x = rng.normal(1, 2, n)
        x[rng.random(n) < 0.01] *= 1e35  # sums stay finite
        return x

    def infinite(n, fr):
        # one a frame, after every state can be reached: all metrics become
        # +inf there and every later decision is a tie
        x = huge(n, fr)
        for k, S in enumerate(lens):
            t = int(rng.integers(code.K, S))
            x[int(fr[k]["llr_offset"]) + t * code.beta] = np.inf if k % 2 else -np.inf
        return x

    _run(code, lens, [1, 0, 3, 2, 1, 3], huge, "f32", variant)
    _run(code, lens, [1, 0, 3, 2, 1, 3], infinite, "f32", variant)


def test_nan_frame_is_deterministic():
    """A frame that holds NaNs ends in a valid state, the same every time, and
    leaves the others alone."""
    rng = np.random.default_rng(20)
    x = rng.normal(1, 2, (4, 300 * 3)).astype(np.float32)
    x[1, 100:110] = np.nan
    outs = []
    for _ in range(3):
        t = torch.from_numpy(x).to("cuda:0")
        w, m = mv.decode(t, CODE_K9, 300, False)
        outs.append((w.cpu().numpy(), m.cpu().numpy()))
    keep = [0, 2, 3]
    ob, om, _ = oracle.decode_uniform(CODE_K9, x[keep], 300, False, oracle.F32)
    for w, m in outs:
        np.testing.assert_array_equal(w, outs[0][0])
        np.testing.assert_array_equal(mv.unpack_bits(w, 300)[keep], ob)
        np.testing.assert_array_equal(m[keep], om)
