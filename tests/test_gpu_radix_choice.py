"""Plans that leave the radix open: int8 K = 5, 7 rate-1/2 parts run the packed
radix-4 kernel except where the frames are few and short.  Either way the
results are those of both explicit radices and of the oracle."""
import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import CODE_K5, CODE_K7, CODE_K9

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _frames(lens, rng, beta=2):
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    off, boff = 3, 0
    for k, S in enumerate(lens):
        n = max(int(S) - int(rng.integers(0, 7)), 0)
        fr[k] = (off, boff, S, 0, n, 0, int(rng.integers(0, 4)))
        off += beta * int(S)
        boff += (n + 31) // 32 * 32
    return fr, off, boff


def _run(code, fr, x, radix, n_bits, **kw):
    plan = mv.Plan([code], fr, "i8", radix, **kw)
    w, m, e = plan.decode(x)
    bits = mv.unpack_bits(w.cpu().numpy(), n_bits)
    got = [bits[int(f["bit_offset"]):int(f["bit_offset"]) + int(f["n_out"])] for f in fr]
    return plan.describe(), np.concatenate(got), m.cpu().numpy(), e.cpu().numpy()


# (lengths, packed by choice): one frame on both sides of the shortest split
# one; counts on both sides of one radix-2 wavefront per SIMD (256 CUs)
CASES = {"short": ([1], False), "odd": ([575, 7, 1], False), "split": ([576], True),
         "long": ([5001, 20], True), "few": ([40] * 1024, False), "many": ([40] * 1100, True)}


@pytest.mark.parametrize("name", list(CASES))
def test_open_radix_k7(name):
    lens, packed = CASES[name]
    rng = np.random.default_rng(len(lens))
    fr, n, n_bits = _frames(lens, rng)
    x = rng.integers(-128, 128, n).astype(np.int8)
    xd = torch.from_numpy(x).to("cuda:0")
    print("open radix", name, flush=True)
    d, b0, m0, e0 = _run(CODE_K7, fr, xd, 0, n_bits)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ("packed" in d) == packed
    for radix in (2, 4):
        _, b, m, e = _run(CODE_K7, fr, xd, radix, n_bits)
        np.testing.assert_array_equal(b0, b)
        np.testing.assert_array_equal(m0, m)
        np.testing.assert_array_equal(e0, e)
    ofr = np.zeros(len(fr), oracle.FRAME_DTYPE)
    for k, f in enumerate(fr):
        ofr[k] = (f["llr_offset"], f["bit_offset"], f["n_stages"], f["out_begin"], f["n_out"],
                  int(f["flags"]) & 1, 0 if int(f["flags"]) & 2 else -1, 0)
    _, om, oe, _ = oracle.decode_frames([CODE_K7], ofr, x, oracle.I64, n_bits)
    np.testing.assert_array_equal(m0, om)
    np.testing.assert_array_equal(e0, oe)


@pytest.mark.parametrize("chunk,overlap", [(512, 64), (96, 30)])
def test_open_radix_chunked(chunk, overlap):
    """Chunks of one long frame: the choice sees the chunks."""
    rng = np.random.default_rng(chunk)
    fr = np.zeros(1, mv.FRAME_DTYPE)
    S = 200001
    fr[0] = (0, 0, S, 0, S, 0, 1)
    xd = torch.from_numpy(rng.integers(-128, 128, 2 * S).astype(np.int8)).to("cuda:0")
    print("open radix chunked", chunk, flush=True)
    for code in (CODE_K5, CODE_K7):
        _, b0, m0, e0 = _run(code, fr, xd, 0, S, chunk=chunk, overlap=overlap)
        for radix in (2, 4):
            _, b, m, e = _run(code, fr, xd, radix, S, chunk=chunk, overlap=overlap)
            np.testing.assert_array_equal(b0, b)
            np.testing.assert_array_equal(m0, m)
            np.testing.assert_array_equal(e0, e)


def test_open_radix_elsewhere_is_two():
    """Options and codes that the packed kernel does not take stay radix 2."""
    fr, _, _ = _frames([3000] * 8, np.random.default_rng(0))
    for kw in ({"variant": 1}, {"variant": 2}, {"persistent": True}):
        assert "packed" not in mv.Plan([CODE_K7], fr, "i8", 0, **kw).describe()
    assert "packed" not in mv.Plan([CODE_K7], fr, "f32", 0).describe()
    assert "radix-2" in mv.Plan([CODE_K9], fr, "i8", 0).describe()
