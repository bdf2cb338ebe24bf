"""GPU tests of the sampling path's kernels at the vocabulary sizes where their
forms change: a thread's share of one entry, chunk lengths odd and even, the
largest row kept in LDS and the first beyond it, one and two slabs of a row in
either width of load.  Decisions against the oracle (inputs redrawn until they
are clear), statistics at the bounds of tests/test_gpu_kernels.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import entmtp_oracle as orc  # noqa: E402
from paper_2606_27550_amd import synth  # noqa: E402
from tests import test_gpu_kernels as kern  # noqa: E402
from tests import test_gpu_speculative as spec  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27550_amd import api as _api
    return _api


@pytest.mark.parametrize("V", [2, 1023, 1025, 30723, 32768, 32769, 50001])
def test_stochastic_vocabulary_sizes(api, V):
    g = np.random.default_rng(V)
    parent = synth.uniform_attach_tree(17, 24, 3)
    for rep in range(3):
        z, q, tok, ua, us, ref = spec.make_inputs(g, parent, V, 1 / 0.7)
        print("[gpu-test] stochastic V", V, "rep", rep, "tests", len(ref[4]) - 1, flush=True)
        a, path, bonus = spec.run(api, parent, z, q, tok, ua, us, 1 / 0.7)
        assert (a, bonus) == (ref[0], ref[2])
        assert path[: a + 1] == list(ref[1])


@pytest.mark.parametrize("V", [1, 3, 4, 2047, 2048, 16384, 16385, 32768, 32772, 65537])
def test_logit_stats_slabs(api, V):
    print("[gpu-test] logit_stats V", V, flush=True)
    g = np.random.default_rng(V)
    z = g.normal(0, 2.5, (3, V)).astype(np.float32)
    z[1, : V // 2] = -np.inf   # masked entries
    z[2, V - 1] = 40.0         # the last entry wins
    kern.check_stats(kern.run_stats(api, z, 1.0), orc.logit_stats(z))
