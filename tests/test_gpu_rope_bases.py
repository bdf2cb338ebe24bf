"""GPU test of the rotation at bases whose largest angle leaves the range of
the short fp64 sine (bases below one turn by more than a radian a position,
past 2^31 radians at ordinary prefixes): cached keys against the same fp64
angles, sines and products from the C library, outputs against float64
attention."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests import test_gpu_attn_plans as plans  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27550_amd import api as _api
    return _api


def turned(x, pos, theta):
    """x [n, H, 128] (float64) at positions pos."""
    ang = [[float(p) * math.pow(theta, -2.0 * c / 128) for c in range(64)] for p in pos]
    cos, sin = (torch.tensor([[f(a) for a in row] for row in ang], dtype=torch.float64,
                             device=x.device)[:, None] for f in (math.cos, math.sin))
    lo, hi = x[..., :64], x[..., 64:]
    return torch.cat((lo * cos - hi * sin, hi * cos + lo * sin), -1)


@pytest.mark.parametrize("theta,L", [(1e6, 900), (1.0, 300), (0.5, 800), (1e-5, 60000), (1e-6, 5000),
                                     (1e-9, 700), (1e-30, 77)])
@pytest.mark.parametrize("form", ["lone", "batch", "device"])
def test_rotation_bases(api, theta, L, form):
    print("[gpu-test] rotation base", theta, L, form, flush=True)
    theta = float(np.float32(theta))   # what the entry point receives
    parent = plans.tree(27)
    T, Hq, Hkv = len(parent), 2, 2
    bank = api.Bank([parent])
    q, k, v = (plans.normal(s, T, 2, 128) for s in (1, 2, 3))
    kc, vc = plans.normal(4, Hkv, L + T, 128), plans.normal(5, Hkv, L + T, 128)
    rk = kc.clone()
    out = torch.full_like(q, float("nan"))
    if form == "lone":
        ws = torch.empty(max(api.tree_attn_workspace(T, Hq, Hkv, 128, L), 256), dtype=torch.uint8, device="cuda")
        api.tree_attn(bank, 0, q, k, v, kc, vc, L, plans.SCALE, theta, out, ws)
    elif form == "batch":
        ws = torch.empty(max(api.tree_attn_batched_workspace(1, T, Hq, Hkv, 128, L), 256), dtype=torch.uint8, device="cuda")
        api.tree_attn_batched(bank, [0], [L], q, k, v, [kc], [vc], plans.SCALE, theta, out, ws)
    else:
        n = api.tree_attn_batched_device_workspace(bank, 1, Hq, Hkv, 128, L + T)
        dev = [torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([0], [L], [0, T])]
        api.tree_attn_batched_device(bank, *dev, q, k, v, [kc], [vc], plans.SCALE, theta, out,
                                     torch.empty(n, dtype=torch.uint8, device="cuda"))
    depth, seen = [0] * T, torch.eye(T, dtype=torch.bool)
    for i in range(1, T):
        depth[i] = depth[parent[i]] + 1
        seen[i] |= seen[parent[i]]
    pos = [L + d for d in depth]
    rk[:, L:] = turned(k.double(), pos, theta).to(torch.bfloat16).transpose(0, 1)
    # the two libraries' sines differ in the last bit: keys agree but for ties
    # of the bf16 rounding
    assert float((kc != rk).float().mean()) < 1e-4
    assert float((kc.double() - rk.double()).abs().max()) <= 2.0 ** -6
    z = torch.stack([turned(q.double(), pos, theta)[:, h].contiguous() @ rk[h].double().t().contiguous()
                     for h in range(Hq)]) * plans.SCALE
    z[:, :, L:] = z[:, :, L:].masked_fill(~seen.cuda(), -math.inf)
    ref = torch.stack([torch.softmax(z[h], 1) @ vc[h].double() for h in range(Hq)], 1)
    assert float((out.double() - ref).abs().max()) <= plans.TOL
