"""decode, decode_stream and ViterbiDecode allocate their outputs without
clearing them: every word and metric has to be written, pad bits included,
whatever the memory held before."""
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


def _dirty():
    """Leaves blocks of small sizes in the allocator's cache, full of ones."""
    keep = [torch.full((n,), -1, dtype=torch.int32, device="cuda:0")
            for n in (1, 64, 128, 512, 4096, 65536) for _ in range(8)]
    del keep


def _padded(bits, n):
    w = np.zeros((bits.shape[0], (n + 31) // 32 * 32), np.uint8)
    w[:, :n] = bits
    return np.packbits(w, axis=1, bitorder="little").view(np.int32)


@pytest.mark.parametrize("dt", ["i8", "f32", "f16"])
@pytest.mark.parametrize("F,n_info", [(1, 1), (3, 31), (2, 33), (5, 95), (0, 40), (4, 0)])
def test_all_words_written(dt, F, n_info):
    rng = np.random.default_rng(F + n_info)
    td = {"i8": torch.int8, "f32": torch.float32, "f16": torch.float16}[dt]
    for code in (CODE_K5, CODE_K7, CODE_K9):
        for term in (True, False):
            S = n_info + (code.K - 1 if term else 0)
            x = rng.integers(-100, 101, (F, code.beta * S)).astype(np.int8)
            xd = torch.from_numpy(x).to("cuda:0").to(td)
            fr = np.zeros(F, oracle.FRAME_DTYPE)
            W = (n_info + 31) // 32
            for f in range(F):
                fr[f] = (f * S * code.beta, f * n_info, S, 0, n_info, 1, 0 if term else -1, 0)
            ob, om = np.zeros(0, np.uint8), np.zeros(F)
            if F and S:
                ob, om, _, _ = oracle.decode_frames([code], fr, x.reshape(-1), oracle.I64, F * n_info)
            want = _padded(np.asarray(ob[: F * n_info]).reshape(F, n_info), n_info) if F else None
            print("outputs", dt, F, n_info, code.K, term, flush=True)
            for radix in (0, 2) if S else (0,):  # plans refuse soft values of no extent
                _dirty()
                bits, metric = mv.decode(xd, code, n_info, term, radix)
                assert bits.shape == (F, W) and metric.shape == (F,)
                if F:
                    np.testing.assert_array_equal(bits.cpu().numpy(), want.reshape(F, W))
                    np.testing.assert_array_equal(metric.cpu().numpy(), om)
            if dt == "f32" and S:
                _dirty()
                bits, metric = mv.ViterbiDecode.apply(xd, code, n_info, term)
                assert bits.shape == (F, W) and metric.shape == (F,)
                if F:
                    np.testing.assert_array_equal(bits.cpu().numpy(), want.reshape(F, W))
                    np.testing.assert_array_equal(metric.cpu().numpy(), om)


@pytest.mark.parametrize("n", [1, 33, 5000])
def test_stream_words_written(n):
    rng = np.random.default_rng(n)
    x = rng.integers(-100, 101, 2 * n).astype(np.int8)
    xd = torch.from_numpy(x).to("cuda:0")
    fr = np.zeros(1, mv.FRAME_DTYPE)
    fr[0] = (0, 0, n, 0, n, 0, mv.MIVIT_START_KNOWN)
    w, _, _ = mv.Plan([CODE_K7], fr, "i8", 2, 1024, 64).decode(xd)
    _dirty()
    got = mv.decode_stream(xd, CODE_K7, n, 1024, 64)
    np.testing.assert_array_equal(got.cpu().numpy(), w.cpu().numpy()[: (n + 31) // 32])
