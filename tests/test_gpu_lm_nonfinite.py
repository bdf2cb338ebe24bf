"""GPU tests of the LM head's statistics where a vocabulary row's logits are not
finite, at a size for every form it has (with 256 CUs: streaming slices,
128 x 128, 256 x 256 and 256 x 128 tiles): a NaN or +inf logit shows in the
statistics (no finite entropy or probability covers it up), and a row masked
to -inf counts for nothing, as in the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import entmtp_oracle as orc  # noqa: E402
from paper_2606_27550_amd import synth  # noqa: E402
from tests import test_gpu_lm_tiled as tiled  # noqa: E402

pytestmark = pytest.mark.gpu

BF_ONE, BF_INF, BF_NEG_INF, BF_NAN = 0x3F80, 0x7F80, 0xFF80, 0x7FC0
FORMS = [(100, 512, 5000), (140, 512, 5000), (385, 512, 17000), (70, 512, 50000), (300, 1024, 66001)]


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27550_amd import api as _api
    return _api


def stats(api, X, w, it):
    """(entropy, top-1 probability, argmax) of hidden rows X with weight w;
    column 0 of the hidden rows is one."""
    T, hid = X.shape
    V = w.shape[0]
    ws = torch.empty(api.stats_partials_bytes(T, hid, V), dtype=torch.uint8, device="cuda")
    H, p1 = torch.empty(T, device="cuda"), torch.empty(T, device="cuda")
    am = torch.empty(T, dtype=torch.int32, device="cuda")
    z = torch.empty((T, V), device="cuda")
    api.verify_logits_partials(tiled.dev_bf16(X), tiled.dev_bf16(w), z, it, ws)
    api.stats_finalize(ws, T, V, it, H, p1, am)
    return z.cpu().numpy(), H.cpu().numpy(), p1.cpu().numpy(), am.cpu().numpy()


def inputs(T, hid, V):
    X, w = synth.hidden_rows(71, T, hid).copy(), synth.lm_head_weight(72, V, hid, std=0.05).copy()
    X[:, 0] = BF_ONE
    return X, w


@pytest.mark.parametrize("T,hid,V", FORMS)
@pytest.mark.parametrize("bits", [BF_NAN, BF_INF])
def test_nan_and_inf_logits_show(api, T, hid, V, bits):
    X, w = inputs(T, hid, V)
    for row in (0, V // 2, V - 1):
        print("[gpu-test] LM head", hex(bits), "row", row, "of", T, hid, V, flush=True)
        wr = w.copy()
        wr[row, 0] = bits
        z, H, p1, am = stats(api, X, wr, 1 / 0.7)
        assert not np.isfinite(z[:, row]).any()
        assert np.isnan(H).all() and np.isnan(p1).all()
        if bits == BF_INF:
            assert (am == row).all()


@pytest.mark.parametrize("T,hid,V", FORMS)
def test_rows_masked_to_minus_inf(api, T, hid, V):
    X, w = inputs(T, hid, V)
    masked = [0, 1, V // 2, V - 1]
    w[masked, 0] = BF_NEG_INF
    print("[gpu-test] LM head masked rows", T, hid, V, flush=True)
    for it in (1.0, 1 / 0.7):
        z, H, p1, am = stats(api, X, w, it)
        assert (z[:, masked] == -np.inf).all() and np.isfinite(np.delete(z, masked, 1)).all()
        rH, rp1, ram = orc.logit_stats(z, it)
        np.testing.assert_array_equal(am, ram)
        assert np.all(np.abs(H - rH) <= tiled.RTOL_STATS * np.abs(rH) + 1e-6)
        assert np.all(np.abs(p1 - rp1) <= tiled.RTOL_STATS * np.abs(rp1) + 1e-6)
