"""int8 rate-1/4 codes of K = 8 and 9, whose metrics do not fit 16 bits: the
32-bit forward with its check and repair launches, and the traceback of its
survivor bytes, against the oracle: stage counts around blocks and phase
periods, every kind of start and end, frames split in time with boundaries that
fail at several places, and the allocation-free call."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2011_13579_amd as mv
from workload import Code, make_uniform_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CODES = [Code.from_octal(8, ["235", "275", "313", "357"]),
         Code.from_octal(9, ["463", "535", "733", "745"])]
# outputs that are all alike: two-state chains, whose boundaries never merge
CHAINS = [Code.from_octal(8, ["201"] * 4), Code.from_octal(9, ["401"] * 4)]
IDS = ["K8", "K9"]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _check(code, lens, flags, llr_of, split=True, out_of=None):
    fr = np.zeros(len(lens), mv.FRAME_DTYPE)
    ofr = np.zeros(len(lens), oracle.FRAME_DTYPE)
    off, boff, parts = 1, 0, []  # soft values at odd addresses
    for k, (S, fl) in enumerate(zip(lens, flags)):
        ob, n = out_of(k, S) if out_of else (0, S)
        fr[k] = (off, boff, S, ob, n, 0, fl)
        ofr[k] = (off, boff, S, ob, n, fl & 1, 0 if fl & 2 else -1, 0)
        parts.append(llr_of(k, S))
        off += 4 * S
        boff += (n + 31) // 32 * 32
    x = np.concatenate([np.zeros(1)] + parts).astype(np.int8)
    print("rate 1/4", code.K, len(lens), split, flush=True)
    plan = mv.Plan([code], fr, "i8", 0, split=split)
    d = plan.describe()
    assert "states in registers" in d and "two states per register" not in d
    w, m, e = plan.decode(torch.from_numpy(x).to("cuda:0"))
    ob, om, oe, _ = oracle.decode_frames([code], ofr, x, oracle.I64, boff)
    np.testing.assert_array_equal(m.cpu().numpy(), om)
    np.testing.assert_array_equal(e.cpu().numpy(), oe)
    got = mv.unpack_bits(w.cpu().numpy(), boff)
    for k in range(len(fr)):
        a, n = int(fr[k]["bit_offset"]), int(fr[k]["n_out"])
        np.testing.assert_array_equal(got[a:a + n], ob[a:a + n])


LENS = [1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 223, 224, 225, 255, 256, 257, 671, 672, 673]


@pytest.mark.parametrize("code", CODES + CHAINS, ids=IDS + ["K8-chain", "K9-chain"])
def test_blocks_and_periods(code):
    rng = np.random.default_rng(19 * code.K)
    flags = rng.integers(0, 4, len(LENS))
    _check(code, LENS, flags, lambda k, S: rng.integers(-128, 128, 4 * S))
    _check(code, LENS, flags, lambda k, S: np.full(4 * S, [-128, 127, 0][k % 3]),
           out_of=lambda k, S: (k % 5 * S // 5, S - k % 5 * S // 5 - k % 2 * (S // 7)))


@pytest.mark.parametrize("code", CODES, ids=IDS)
@pytest.mark.parametrize("noise", ["0dB", "none but noise", "ties"])
def test_split_in_time(code, noise):
    """511 stages stay whole, 1024 are cut in two, the longest in eight."""
    rng = np.random.default_rng(23 * code.K)
    lens = [511, 1024, 1025, 3001, 5000, 9003]

    def llr(k, S):
        if noise == "0dB":
            b = make_uniform_batch(code, 1, S, 0.0, seed=k, terminated=False)
            return oracle.quantize_i8(b.llr[0], 8.0)
        return rng.integers(-128, 128, 4 * S) if noise != "ties" else np.zeros(4 * S)

    x = [llr(k, S) for k, S in enumerate(lens)]
    for split in (True, False):
        _check(code, lens, [0, 1, 2, 3, 1, 0], lambda k, S: x[k], split)


@pytest.mark.parametrize("code", CHAINS, ids=IDS)
def test_boundaries_that_never_merge(code):
    rng = np.random.default_rng(29)
    S = 6001
    x = [np.full(4 * S, 100), np.repeat(rng.choice([-90, 90], S), 4),
         np.repeat(rng.choice([-128, 127], S), 4)]
    _check(code, [S] * 3, [1, 3, 0], lambda k, n: x[k])


@pytest.mark.parametrize("code", CODES, ids=IDS)
def test_allocation_free_call(code):
    F, n = 9, 701
    rng = np.random.default_rng(31)
    x = rng.integers(-128, 128, (F, 4 * (n + code.K - 1))).astype(np.int8)
    t = torch.from_numpy(x).to("cuda:0")
    bits = torch.full((F * ((n + 31) // 32),), -1, dtype=torch.int32, device="cuda:0")
    metric = torch.zeros(F, dtype=torch.int64, device="cuda:0")
    cs = mv.Code(code.K, tuple(code.gens)).c_struct()
    st = mv._capi.load().mivit_decode_uniform_noalloc(
        t.data_ptr(), mv.MIVIT_I8, ctypes.byref(cs), F, n, 1, bits.data_ptr(), metric.data_ptr(),
        torch.cuda.current_stream().cuda_stream)
    assert st == mv._capi.MIVIT_OK
    ob, om, _ = oracle.decode_uniform(code, x, n, True, oracle.I64)
    np.testing.assert_array_equal(mv.unpack_bits(bits.cpu().numpy().reshape(F, -1), n), ob)
    np.testing.assert_array_equal(metric.cpu().numpy(), om)
