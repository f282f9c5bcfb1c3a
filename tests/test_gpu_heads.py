"""The Gram form with one workgroup per head, which calls of two or more
iterations run: against the float64 oracle and against the sweeps (forced by
explicit strip counts) at the edges of its tiles, slots and launch shapes."""

import numpy as np
import pytest
import torch

from oracle.power_iteration import spectral_step as oracle_step
from workloads import WORKLOADS, all_weights, start_vectors

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2602_18851_amd import Spectral  # noqa: E402
from paper_2602_18851_amd import spectral as sp  # noqa: E402

# sigma: fp32 sums, about 1e-7; vectors: the grouped key products split fp32
# vectors into two bf16 halves (2^-17 = 8e-6), which a head whose two largest
# singular values lie close together can carry on a few times larger.  The
# sweeps take sigma itself through such halves (twice per step), and at d = 1
# no sum over columns averages their errors.
SIGMA_TOL, VEC_TOL, SWEEP_SIGMA_TOL = 2e-6, 1e-4, 2e-5

CASES = [
    # (id, layers, d, pad, n_kv, group, d_h, dtype)
    ("one-tile", 1, 64, 0, 2, 1, 64, "bf16"),                 # one whole tile
    ("one-column", 1, 1, 7, 2, 3, 64, "bf16"),                # a single column, ragged only
    ("tile-and-one", 1, 65, 7, 2, 2, 32, "bf16"),             # unaligned rows of v: 4-byte loads
    ("dh16-f32-17-heads", 1, 100, 0, 2, 17, 16, "f32"),       # two z0 operands of 16 heads
    ("dh16-bf16", 2, 333, 3, 3, 1, 16, "bf16"),
    ("dh32-6-heads", 1, 200, 0, 2, 6, 32, "bf16"),            # three parts: 5 + 1 heads
    ("dh64-9-heads", 1, 1001, 7, 2, 9, 64, "bf16"),           # two parts: 8 + 1 heads
    ("dh128-8-heads", 2, 1000, 0, 3, 8, 128, "bf16"),
    ("dh128-f32", 1, 1003, 1, 2, 2, 128, "f32"),              # unaligned rows of v
    ("own-dh128", 2, 136, 0, 128, 1, 128, "bf16"),            # 256 heads: Q and K by one workgroup
    ("own-dh64-f32", 4, 203, 1, 65, 1, 64, "f32"),
    ("keys-dh64", 4, 200, 0, 32, 2, 64, "bf16"),              # 256 heads: Q by one workgroup, K by another
    ("keys-dh32-f32", 2, 257, 3, 9, 16, 32, "f32"),
    ("keys-dh128-chunks", 4, 64, 0, 480, 2, 128, "bf16"),     # more key heads than one launch pair takes
    # d_h 16, where two of the four waves request no rows, and ten or more tiles per strip
    ("dh16-own-10-tiles", 2, 640, 0, 128, 1, 16, "bf16"),
    ("dh16-own-11-tiles-f32", 2, 331, 1, 128, 1, 16, "f32"),      # unaligned rows of v
    ("dh16-5-heads-10-tiles", 1, 4480, 0, 50, 5, 16, "bf16"),     # 7 strips; wave 3 requests start vectors too
    ("dh16-5-heads-11-tiles", 1, 4483, 5, 50, 5, 16, "bf16"),     # unaligned rows of v
    ("dh16-12-heads-10-tiles-f32", 1, 6080, 0, 20, 12, 16, "f32"),
]


def _workload(layers, d, n_kv, group, dh, dtype, n_iter=6):
    return WORKLOADS["llama2-70b-gqa"].replace(key="heads", cfg_id=77, n_layers=layers, d_model=d, n_q=n_kv * group,
                                               n_kv=n_kv, head_dim=dh, dtype=dtype, n_iter=n_iter, std=0.02)


def _padded(w, pad):
    if not pad:
        return w.cuda()
    p = torch.full((*w.shape[:2], w.shape[2] + pad), float("nan"), dtype=w.dtype)  # columns past d are never used
    p[:, :, :w.shape[2]] = w
    return p.cuda()[:, :, :w.shape[2]]


def _run(wl, wq, wk, v0, ld=0, **kw):
    est = Spectral(wl.n_layers, wl.d_model, wl.n_q, wl.n_kv, wl.head_dim, wl.dtype, wl.alpha, ld=ld, **kw)
    v = v0.cuda().clone()
    u = torch.empty_like(v)
    sigma, scale, iters = est.step(wq, wk, v, wl.n_iter, u=u)
    torch.cuda.synchronize()
    est.close()
    return {k: t.cpu().double().numpy() for k, t in
            dict(sigma=sigma, scale=scale, iters=iters, v=v, u=u).items()}


def _check(got, ref, what, sigma_tol=SIGMA_TOL, vec_tol=VEC_TOL):
    np.testing.assert_array_equal(got["iters"], ref["iters"], err_msg=what)
    for k, tol in (("sigma", sigma_tol), ("scale", sigma_tol)):
        err = np.max(np.abs(got[k] - ref[k]) / np.abs(ref[k]))
        assert err <= tol, (what, k, err)
    for k in ("v", "u"):
        err = np.linalg.norm(got[k] - ref[k], axis=-1).max()
        assert err <= vec_tol, (what, k, err)


@pytest.mark.parametrize("layers,d,pad,n_kv,group,dh,dtype", [c[1:] for c in CASES], ids=[c[0] for c in CASES])
def test_heads_against_oracle_and_sweeps(layers, d, pad, n_kv, group, dh, dtype):
    wl = _workload(layers, d, n_kv, group, dh, dtype)
    wq, wk = all_weights(wl, "cpu")
    v0 = start_vectors(wl, "cpu")
    gq, gk, ld = _padded(wq, pad), _padded(wk, pad), d + pad
    ref = oracle_step(wq.float().numpy(), wk.float().numpy(), v0.double().numpy(), wl.n_iter, n_kv=n_kv, head_dim=dh,
                      alpha=wl.alpha, want_u=True)
    heads = _run(wl, gq, gk, v0, ld)
    _check(heads, ref, "heads")
    _check(_run(wl, gq, gk, v0, ld, q_strips=1, k_strips=1), heads, "sweeps", SWEEP_SIGMA_TOL)


@pytest.mark.parametrize("layers,n_kv,group", [(1, 2, 2), (4, 65, 1), (4, 33, 2)], ids=["split", "own", "keys"])
def test_cancelling_rows(layers, n_kv, group):
    """Rows that share a large common part, which key rows summing to zero make
    cancel in Q^T z: sigma^2 = z^T G_Q z loses all its digits in fp32 (shown
    here with exact Gram matrices), so these heads have to be iterated on the
    weights.  There Q^T z rounds at 6e-8 of the common part, about 1e-4 of
    sigma (the common part is 1e3 times the rest)."""
    dh, d = 16, 96
    wl = _workload(layers, d, n_kv, group, dh, "f32", n_iter=4)
    wq, wk = all_weights(wl, "cpu")
    g = torch.Generator().manual_seed(5)
    common = torch.randn(layers, n_kv * group, 1, d, generator=g) * 20.0
    wq = (wq.view(layers, -1, dh, d) + common).reshape(wq.shape)
    wk = wk.view(layers, n_kv, dh, d)
    wk = (wk - wk.double().mean(dim=2, keepdim=True).float()).reshape(layers, n_kv * dh, d)
    v0 = start_vectors(wl, "cpu")
    qd, kd = wq[0, :dh].double().numpy(), wk[0, :dh].double().numpy()
    z = kd @ v0[0, 0].double().numpy()
    g32, z32 = (qd @ qd.T).astype(np.float32), z.astype(np.float32)
    gram, true = float(z32 @ (g32 @ z32)), float(np.sum((qd.T @ z) ** 2))
    assert abs(gram - true) > 0.1 * true
    ref = oracle_step(wq.numpy(), wk.numpy(), v0.double().numpy(), wl.n_iter, n_kv=n_kv, head_dim=dh, alpha=wl.alpha,
                      want_u=True)
    gq, gk = wq.cuda(), wk.cuda()
    _check(_run(wl, gq, gk, v0, q_strips=1, k_strips=1), ref, "sweeps", 1e-3, 5e-3)
    _check(_run(wl, gq, gk, v0), ref, "heads", 1e-3, 5e-3)


def _correlated(n_q, n_kv, dh, d, dtype, common):
    """Query rows of a head share a part of `common` times their own size, and
    key rows sum to zero, so that Q^T z loses the common part in every step."""
    g = torch.Generator().manual_seed(11)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.randn(n_q, dh, d, generator=g) * 0.02 + torch.randn(n_q, 1, d, generator=g) * (0.02 * common)
    k = torch.randn(n_kv, dh, d, generator=g) * 0.02
    k -= k.mean(dim=1, keepdim=True)
    return q.to(dt).cuda(), k.to(dt).cuda(), torch.randn(n_q, d, generator=g).cuda()


def _chain64(q, k, v, n):
    """sigma and v of every head after n steps through the weights in float64."""
    q, k = q.double(), k.double().repeat_interleave(q.shape[0] // k.shape[0], dim=0)
    qt, kt = q.transpose(1, 2).contiguous(), k.transpose(1, 2).contiguous()
    v = v.double().unsqueeze(2)
    v = v / torch.linalg.vector_norm(v, dim=1, keepdim=True)
    for _ in range(n):
        u = torch.bmm(qt, torch.bmm(k, v))
        sigma = torch.linalg.vector_norm(u, dim=1, keepdim=True)
        v = torch.bmm(kt, torch.bmm(q, u / sigma))
        v = v / torch.linalg.vector_norm(v, dim=1, keepdim=True)
    return sigma.flatten(), v.squeeze(2)


CORRELATED = [
    # (id, n_q, n_kv, d_h, d, dtype): one per way of iterating (rows, blocks, float under bf16 halves) and type
    ("dh16-f32", 96, 96, 16, 768, "f32"),
    ("dh64-f32", 144, 144, 64, 768, "f32"),
    ("dh64-bf16-own", 300, 300, 64, 768, "bf16"),
    ("dh128-f32", 64, 64, 128, 1024, "f32"),
    ("dh128-bf16", 64, 64, 128, 1024, "bf16"),
    ("dh128-bf16-own", 300, 300, 128, 512, "bf16"),
    ("dh128-f32-keys", 300, 150, 128, 512, "f32"),
    ("dh128-halves", 64, 8, 128, 4096, "bf16"),
    ("dh64-halves", 48, 4, 64, 3000, "bf16"),
]


@pytest.mark.parametrize("common", [0.0, 0.9, 1.7, 3.4])
@pytest.mark.parametrize("n_q,n_kv,dh,d,dtype", [c[1:] for c in CORRELATED], ids=[c[0] for c in CORRELATED])
def test_no_less_precise_than_the_sweeps(n_q, n_kv, dh, d, dtype, common):
    """Over heads whose rows cancel to sigma^2 / b = 1, 0.55, 0.25 and 0.08 (b =
    sum_i z_i^2 ||q_i||^2): the rms error of v against float64, and that of sigma
    beside its own rounding to 32 bits (6e-8), are at most those of the sweeps."""
    q, k, v0 = _correlated(n_q, n_kv, dh, d, dtype, common)
    s64, v64 = _chain64(q, k, v0, 20)
    err = {}
    for form, strips in (("sweeps", 1), ("heads", 0)):
        est = Spectral(1, d, n_q, n_kv, dh, dtype, 0.05, q_strips=strips, k_strips=strips)
        v = v0.clone().unsqueeze(0)
        sigma, _, _ = est.step(q.reshape(1, -1, d), k.reshape(1, -1, d), v, 20)
        torch.cuda.synchronize()
        est.close()
        err[form] = [((sigma[0].double() - s64) / s64).square().mean().sqrt().item(),
                     (v[0].double() - v64).square().sum(dim=1).mean().sqrt().item()]
    print(err)
    assert err["heads"][1] <= err["sweeps"][1], err
    assert err["heads"][0] <= max(err["sweeps"][0], 8e-8), err


@pytest.mark.parametrize("n_q,n_kv,dh,d,dtype,spread",
                         [(300, 300, 64, 1600, "bf16", 0.0), (64, 64, 128, 2048, "bf16", 0.0),
                          (64, 8, 128, 4096, "bf16", 0.0), (96, 96, 16, 768, "f32", 1.0)],
                         ids=["rows", "blocks", "halves", "uneven-rows"])
def test_passing_cancellation_stays_in_dh_space(n_q, n_kv, dh, d, dtype, spread):
    """Query rows with a large common part and a random start: some heads cancel
    in their first step alone (the smallest sigma^2 / b here is 0.2), and rows of
    uneven size leave ||G z|| small against its bound.  Neither loses precision
    against the sweeps, and neither may send a head to its weights, which would
    take several times as long."""
    g = torch.Generator().manual_seed(3)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def weights(common):
        q = (torch.randn(n_q, dh, d, generator=g) + common * torch.randn(n_q, 1, d, generator=g)) * 0.02
        k = torch.randn(n_kv, dh, d, generator=g) * 0.02
        q *= 10 ** (spread * (2 * torch.rand(n_q, dh, 1, generator=g) - 1))
        k *= 10 ** (spread * (2 * torch.rand(n_kv, dh, 1, generator=g) - 1))
        return q.to(dt).cuda(), k.to(dt).cuda()

    v0 = torch.randn(n_q, d, generator=g).cuda()

    def run(q, k, strips):
        est = Spectral(1, d, n_q, n_kv, dh, dtype, 0.05, q_strips=strips, k_strips=strips)
        times = []
        for _ in range(5):
            v = v0.clone().unsqueeze(0)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            est.step(q.reshape(1, -1, d), k.reshape(1, -1, d), v, 20)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        est.close()
        return v[0].double(), sorted(times)[2]

    q, k = weights(2.0)
    _, v64 = _chain64(q, k, v0, 20)
    err = {strips: (run(q, k, strips)[0] - v64).square().sum(dim=1).mean().sqrt().item() for strips in (1, 0)}
    assert err[0] <= err[1], err
    plain = run(*weights(0.0 if spread == 0 else 0.5), 0)[1]
    assert run(q, k, 0)[1] <= 2 * plain


def test_zero_rows():
    """Rows of zeros (pruned or padded dimensions of a head) keep the form's
    results and its speed: 300 steps on the weights instead of in d_h-space would
    take many times as long."""
    wl = _workload(4, 1024, 64, 1, 64, "bf16", n_iter=6)
    wq, wk = all_weights(wl, "cpu")
    v0 = start_vectors(wl, "cpu")
    zq, zk = wq.clone().view(4, 64, 64, 1024), wk.clone().view(4, 64, 64, 1024)
    zq[:, :, 40:48], zk[:, ::2, 60:] = 0, 0
    zq[1, 3], zk[2, 5] = 0, 0      # and whole heads: M = 0
    zq, zk = zq.reshape(wq.shape), zk.reshape(wk.shape)
    ref = oracle_step(zq.float().numpy(), zk.float().numpy(), v0.double().numpy(), wl.n_iter, n_kv=wl.n_kv, head_dim=64,
                      alpha=wl.alpha, want_u=True)
    got = _run(wl, zq.cuda(), zk.cuda(), v0)
    np.testing.assert_array_equal(got["iters"], ref["iters"])
    assert got["iters"][1, 3] == got["iters"][2, 5] == -2
    live = ref["iters"] > 0
    assert np.max(np.abs(got["sigma"] - ref["sigma"])[live] / ref["sigma"][live]) <= SIGMA_TOL
    for x in ("v", "u"):
        assert np.linalg.norm(got[x] - ref[x], axis=-1).max() <= VEC_TOL

    def step_time(q, k):
        est = Spectral(4, 1024, 64, 64, 64, "bf16", wl.alpha)
        q, k, v = q.cuda(), k.cuda(), v0.cuda()
        est.step(q, k, v, 300)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        est.step(q, k, v, 300)
        b.record()
        torch.cuda.synchronize()
        est.close()
        return a.elapsed_time(b)

    dense, zeros = step_time(wq, wk), step_time(zq, zk)
    print(f"300 steps: {dense:.3f} ms, with zero rows {zeros:.3f} ms")
    assert zeros <= 2 * dense


def test_values_outside_the_range_of_gram_products():
    """Query weights near 1e-20 and key weights near 1e18: the products in G_Q
    underflow, those in G_K overflow, and u' = Q^T z is an ordinary number."""
    wl = _workload(2, 200, 2, 2, 32, "f32")
    wq, wk = all_weights(wl, "cpu")
    wq, wk = wq * 2.0 ** -60, wk * 2.0 ** 66
    v0 = start_vectors(wl, "cpu")
    ref = oracle_step(wq.numpy(), wk.numpy(), v0.double().numpy(), wl.n_iter, n_kv=2, head_dim=32, alpha=wl.alpha,
                      want_u=True)
    _check(_run(wl, wq.cuda(), wk.cuda(), v0), ref, "heads")


NOALLOC_CASES = [
    # (id, layers, d, n_kv, group, d_h, dtype): 8 to 66 tiles per strip, so that a head's tile order shows
    ("pairs", 4, 512, 240, 2, 128, "bf16"),                # Gram matrices of 960 key heads: more than the scratch
    ("pairs-8-heads", 30, 1024, 32, 8, 128, "bf16"),
    ("one-key-head", 1, 16384, 1, 8, 128, "bf16"),         # split into strips; a single unit takes most of the scratch
    ("one-wide-key-head", 1, 65536, 1, 8, 128, "bf16"),
    ("split", 2, 2112, 3, 4, 64, "f32"),
]


@pytest.mark.parametrize("layers,d,n_kv,group,dh,dtype", [c[1:] for c in NOALLOC_CASES],
                         ids=[c[0] for c in NOALLOC_CASES])
def test_noalloc_gives_the_same_bits(layers, d, n_kv, group, dh, dtype):
    """The static scratch leaves room for fewer key heads per launch pair than
    a context, down to one; the results do not depend on it."""
    wl = _workload(layers, d, n_kv, group, dh, dtype)
    gq, gk = all_weights(wl, "cuda")
    v0 = start_vectors(wl, "cuda")
    ref = _run(wl, gq, gk, v0)
    v, u = v0.clone(), torch.empty_like(v0)
    sigma = torch.empty(wl.n_layers, wl.n_q, device="cuda")
    scale, iters = torch.empty(wl.n_layers, device="cuda"), torch.empty(sigma.shape, dtype=torch.int32, device="cuda")
    shape = sp.sn_shape(wl.n_layers, wl.d_model, wl.n_q, wl.n_kv, wl.head_dim,
                        sp.SN_BF16 if dtype == "bf16" else sp.SN_F32, 0)
    sp.spectral_step_noalloc(shape, sp.sn_params(wl.alpha, 0.8, 448.0, 0.0, 0, 0, 0),
                             [t.data_ptr() for t in gq.unbind(0)], [t.data_ptr() for t in gk.unbind(0)], v.data_ptr(),
                             u.data_ptr(), wl.n_iter, sigma.data_ptr(), scale.data_ptr(), iters.data_ptr(),
                             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for k, t in dict(v=v, u=u, sigma=sigma, scale=scale, iters=iters).items():
        np.testing.assert_array_equal(t.cpu().double().numpy(), ref[k], err_msg=k)


def test_context_of_several_launch_pairs():
    """More key heads than one launch pair takes: the launch counts say so, and
    the heads of each pair agree with the same heads in a context of their own."""
    wl = _workload(4, 512, 480, 2, 128, "bf16", n_iter=3)
    gq, gk = all_weights(wl, "cuda")
    v0 = start_vectors(wl, "cuda")
    est = Spectral(wl.n_layers, wl.d_model, wl.n_q, wl.n_kv, wl.head_dim, wl.dtype, wl.alpha)
    est.profile(True)
    v = v0.clone()
    sigma, _, _ = est.step(gq, gk, v, wl.n_iter)
    torch.cuda.synchronize()
    prof = est.profile_read()
    est.close()
    assert prof["gram_sweep"][1] == prof["gram_iterate"][1] >= 2, prof
    for l in range(wl.n_layers):
        one = _run(wl.replace(n_layers=1), gq[l:l + 1], gk[l:l + 1], v0[l:l + 1])
        # another layer count may take other column strips and another tile order
        np.testing.assert_allclose(sigma[l].cpu().double().numpy(), one["sigma"][0], rtol=SIGMA_TOL)
        assert np.linalg.norm(v[l].cpu().double().numpy() - one["v"][0], axis=-1).max() <= VEC_TOL


def test_tolerance_calls_over_64_mib_of_weights():
    """Large tolerance calls iterate in the per-head kernel: the stop of every
    head against the oracle's own sequence (10% of the threshold, the precision
    of the difference of two estimates), and its vectors at that step."""
    from oracle.power_iteration import head_slices, power_iteration

    wl = WORKLOADS["llama2-70b-perstep"].replace(key="tol-heads", cfg_id=78, n_layers=2, d_model=2048, n_q=64, n_kv=8)
    assert sum(wl.weight_bytes()) >= 64 << 20
    wq, wk = all_weights(wl, "cpu")
    v0 = start_vectors(wl, "cpu")
    est = Spectral(wl.n_layers, wl.d_model, wl.n_q, wl.n_kv, wl.head_dim, wl.dtype, wl.alpha, tol=wl.tol)
    v = v0.cuda()
    est.profile(True)
    sigma, _, iters = est.step(wq.cuda(), wk.cuda(), v, wl.n_iter)
    torch.cuda.synchronize()
    prof = est.profile_read()
    est.close()
    assert prof["q_sweep"][1] == 0 and prof["gram_iterate"][1] == 1
    it, sig, vv = iters.cpu().numpy(), sigma.cpu().double().numpy(), v.cpu().double().numpy()
    wqf, wkf = wq.float().numpy(), wk.float().numpy()
    for l in range(wl.n_layers):
        for h in range(0, wl.n_q, 5):
            q, k = head_slices(wqf[l], wkf[l], h, wl.n_kv, wl.head_dim)
            n = int(it[l, h])
            r = power_iteration(q, k, v0[l, h].double().numpy(), n)
            change = [abs(b - a) / (wl.tol * b) for a, b in zip(r.history, r.history[1:])]
            assert n >= 2 and change[-1] <= 1.1 and min(change[:-1], default=1.0) >= 0.9, (l, h, n)
            assert abs(sig[l, h] - r.sigma) <= SIGMA_TOL * r.sigma
            assert np.linalg.norm(vv[l, h] - r.v) <= VEC_TOL
