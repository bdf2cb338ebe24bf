"""GPU parity of the tiled LM head at hidden sizes of every stage count's
remainder, with ragged batches and vocabularies of odd size (rows of logits at
any multiple of four bytes), against the oracle at the bounds of
tests/test_gpu_lm_tiled.py.  The forms as 256 CUs dispatch them: 128 x 128
tiles (rounds of four stages, of which a multiple of 512 leaves none), 256 x 256
and 256 x 128 tiles (rounds of six: none, two or four left; the last with three
live 16-row blocks of X too)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2606_27550_amd import synth  # noqa: E402
from tests import test_gpu_lm_tiled as tiled  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27550_amd import api as _api
    return _api


@pytest.mark.parametrize("T,hid,V", [
    (129, 512, 16385), (140, 1024, 1027), (65, 1536, 33001), (257, 2048, 16386), (200, 512, 66001),
    (256, 3584, 4099), (385, 1024, 17000),
    (385, 512, 17000), (400, 1536, 17001),                                          # 256 x 256
    (70, 512, 50001), (110, 1024, 50001), (130, 1536, 50001), (300, 1024, 66001),   # 256 x 128
])
def test_tiled_hidden_sizes(api, T, hid, V):
    print("[gpu-test] tiled LM head", T, hid, V, flush=True)
    w = synth.lm_head_weight(60 + hid // 512, V, hid, std=0.05)
    tiled.check_rows(api, synth.hidden_rows(61, T, hid), w, tiled.dev_bf16(w))
