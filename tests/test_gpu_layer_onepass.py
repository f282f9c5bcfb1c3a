"""One-pass sweeps of the layer-level form (a layer's grouped rows in one
workgroup) against the float64 oracle at the edges of their tiles, waves and
chunks.  Sums are fp32 throughout: sigma to 2e-6, and unit vectors to 2e-5 (a
layer whose two largest singular values lie close together carries a rounding
error on some ten times larger)."""

import numpy as np
import pytest
import torch

from oracle.power_iteration import power_iteration_layer
from workloads import WORKLOADS, all_weights, layer_start_vectors

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2602_18851_amd import SN_FLAG_LAYER, Spectral  # noqa: E402

CASES = [
    # (id, layers, d, pad, n_kv, group, d_h, dtype, n_iter)
    ("1024-rows", 2, 520, 0, 8, 2, 128, "bf16", 4),           # 16 full waves
    ("1024-rows-mha", 1, 256, 0, 8, 1, 128, "bf16", 4),
    ("over-1024-rows", 2, 300, 4, 9, 2, 128, "bf16", 4),      # two passes per sweep, as before
    ("part-of-a-wave", 2, 333, 3, 5, 3, 8, "bf16", 4),        # 40 rows, ragged columns
    ("one-column", 1, 1, 3, 2, 2, 64, "f32", 3),
    ("one-iteration", 2, 200, 0, 3, 4, 64, "bf16", 1),
    ("one-iteration-g2", 2, 200, 0, 3, 2, 64, "bf16", 1),     # group sums would cost more than they save
    ("f32-group", 3, 1003, 1, 2, 12, 32, "f32", 5),
    ("two-chunks", 3, 98304, 0, 8, 2, 128, "bf16", 2),        # group sums of 403 MB a layer: two layers at a time
]


@pytest.mark.parametrize("layers,d,pad,n_kv,group,dh,dtype,n_iter", [c[1:] for c in CASES], ids=[c[0] for c in CASES])
def test_layer_form(layers, d, pad, n_kv, group, dh, dtype, n_iter):
    wl = WORKLOADS["llama2-70b-gqa"].replace(key="onepass", cfg_id=91, n_layers=layers, d_model=d, n_q=n_kv * group,
                                             n_kv=n_kv, head_dim=dh, dtype=dtype, std=0.02)
    wq, wk = all_weights(wl, "cuda" if d > 10000 else "cpu")
    v0 = layer_start_vectors(wl, "cpu")

    def padded(w):
        if not pad:
            return w.cuda()
        p = torch.full((*w.shape[:2], d + pad), float("nan"), dtype=w.dtype)   # columns past d are never used
        p[:, :, :d] = w
        return p.cuda()[:, :, :d]

    est = Spectral(layers, d, wl.n_q, n_kv, dh, dtype, wl.alpha, ld=d + pad, flags=SN_FLAG_LAYER)
    v = v0.cuda().clone()
    u = torch.empty_like(v)
    sigma, _ = est.step_layer(padded(wq), padded(wk), v, n_iter, u=u)
    torch.cuda.synchronize()
    est.close()
    sigma, v, u = (t.cpu().double().numpy() for t in (sigma, v, u))
    for l in range(layers) if d <= 10000 else (1, 2):   # of the wide case one layer of each chunk
        r = power_iteration_layer(wq[l].float().cpu().numpy().T, wk[l].float().cpu().numpy().T,
                                  v0[l].double().numpy(), n_iter, group, dh)
        assert abs(sigma[l] - r.sigma) <= 2e-6 * r.sigma, (l, sigma[l], r.sigma)
        assert np.linalg.norm(v[l] - r.v) <= 2e-5 and np.linalg.norm(u[l] - r.u) <= 2e-5, l


@pytest.mark.parametrize("d,n_q,n_kv,dh", [(200, 8, 2, 32), (328, 32, 8, 128)], ids=["64-rows", "1024-rows"])
def test_degenerate_layers(d, n_q, n_kv, dh):
    """A zero and a non-finite start vector, and key rows whose group has M v =
    0, beside a regular layer: statuses as in the two-pass form."""
    wl = WORKLOADS["llama2-70b-gqa"].replace(key="onepass-degenerate", cfg_id=92, n_layers=4, d_model=d, n_q=n_q,
                                             n_kv=n_kv, head_dim=dh, std=0.02)
    wq, wk = all_weights(wl, "cpu")
    wk[2] = 0
    v0 = layer_start_vectors(wl, "cpu") * 3.0
    v0[0], v0[1, 7] = 0.0, float("inf")
    est = Spectral(4, d, n_q, n_kv, dh, "bf16", wl.alpha, flags=SN_FLAG_LAYER)
    v = v0.cuda().clone()
    u = torch.full_like(v, 7.0)
    sigma, scale = (t.cpu().numpy() for t in est.step_layer(wq.cuda(), wk.cuda(), v, 4, u=u))
    est.close()
    v, u = v.cpu().numpy(), u.cpu().numpy()
    assert np.isnan(sigma[:2]).all() and np.isnan(scale[:2]).all() and sigma[2] == 0 and scale[2] == 0
    np.testing.assert_array_equal(v[:2], v0[:2].numpy())
    np.testing.assert_allclose(v[2], v0[2].numpy() / np.linalg.norm(v0[2].double().numpy()), atol=1e-6)
    assert not u[:3].any()
    r = power_iteration_layer(wq[3].float().numpy().T, wk[3].float().numpy().T, v0[3].double().numpy(), 4, 4, dh)
    assert abs(sigma[3] - r.sigma) <= 2e-6 * r.sigma and np.linalg.norm(v[3] - r.v) <= 2e-5


def test_without_room_for_the_group_sums():
    """A context that cannot have the group sums' 805 MB goes without them."""
    layers, d, n_kv, group, dh = 2, 98304, 8, 2, 128
    wl = WORKLOADS["llama2-70b-gqa"].replace(key="onepass-room", cfg_id=93, n_layers=layers, d_model=d, n_q=n_kv * group,
                                             n_kv=n_kv, head_dim=dh, std=0.02)
    wq, wk = all_weights(wl, "cuda")
    v0 = layer_start_vectors(wl, "cpu").cuda()

    def run():
        est = Spectral(layers, d, wl.n_q, n_kv, dh, "bf16", wl.alpha, flags=SN_FLAG_LAYER)
        v = v0.clone()
        sigma, _ = est.step_layer(wq, wk, v, 2)
        torch.cuda.synchronize()
        est.close()
        return sigma.cpu().double(), v.cpu().double()

    want = run()
    torch.cuda.empty_cache()
    fill, room = [], 600 << 20   # between the 62 MB the context needs and the 867 MB it asks for first
    while (free := torch.cuda.mem_get_info()[0]) > room + (64 << 20):
        fill.append(torch.empty(free - room, dtype=torch.uint8, device="cuda"))
    got = run()
    del fill
    torch.cuda.empty_cache()
    assert ((got[0] - want[0]).abs() <= 2e-6 * want[0]).all()
    assert torch.linalg.vector_norm(got[1] - want[1], dim=1).max() <= 2e-5
