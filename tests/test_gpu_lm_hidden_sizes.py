"""GPU parity of the tiled LM head at hidden sizes whose stage counts leave
each remainder of its six-stage round (multiples of 512: two, four or none),
with ragged batches and vocabularies of odd size (rows of logits at any
multiple of four bytes), against the oracle at the bounds of
tests/test_gpu_lm_tiled.py."""
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
])
def test_tiled_hidden_sizes(api, T, hid, V):
    print("[gpu-test] tiled LM head", T, hid, V, flush=True)
    w = synth.lm_head_weight(60 + hid // 512, V, hid, std=0.05)
    tiled.check_rows(api, synth.hidden_rows(61, T, hid), w, tiled.dev_bf16(w))
