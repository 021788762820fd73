"""Launches of few packets, where a packet's leaves are dealt out to the waves
of a workgroup: against the FP64 oracle, and against the launches that run a
packet on one wave (the per-ray FP64 sum is taken in another order there, so an
FP32 result may differ in its last bit)."""
import numpy as np
import pytest

import oracle
from oracle import geometry as G
from paper_2602_01057_amd.inputs import sample_scene, sample_unit_weights
from parity import assert_forward, assert_grad, gpu_grad_rows
from test_gpu_tof import assert_bins

pytestmark = pytest.mark.gpu

LAST_BIT = 1.2e-7


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# (Gaussians, leaf size, views, nu, nv): one leaf (no parts), as many leaves as parts and one more or less,
# one ragged packet, packets of several runs, and more packets than workgroups take at once
@pytest.mark.parametrize("n,leaf,views,nu,nv", [(50, 64, 1, 8, 8), (130, 64, 1, 5, 7), (15 * 16, 16, 2, 8, 8),
                                                (17 * 16 - 3, 16, 3, 19, 11), (400, 1, 2, 16, 8),
                                                (1500, 8, 5, 33, 21), (900, 64, 40, 40, 24)])
def test_parts_against_oracle_and_whole_packets(gr, n, leaf, views, nu, nv):
    import torch
    sc = sample_scene(n, seed=31 + n, radius=60.0, scale_range=(1.0, 9.0))
    g = dict(kind="ct", cone=1, n_views=views, nu=nu, nv=nv, angle0=0.1, angle_range=5.0, dso=400.0, dsd=700.0,
             pitch_u=190.0 / nu, pitch_v=190.0 / nv, offset_u=0.0, offset_v=0.0, tile_u=8, tile_v=8)
    o, d = G.rays32(g)
    m = o.shape[1]
    S = gr.Scene(*[_dev(a) for a in (sc.mean, sc.scale, sc.quat, sc.density)], leaf_size=leaf)
    ro, rd = _dev(o), _dev(d)
    ref = oracle.project(sc, o, d)
    near = lambda a, b: torch.allclose(a, b, rtol=LAST_BIT, atol=0.0)  # noqa: E731
    I = gr.project(S, ro, rd)
    assert_forward(I.cpu().numpy(), ref, what="parts")
    for kw in (dict(waves_per_group=2), dict(persistent=True), dict(traversal=1), dict(traversal=1, persistent=3)):
        assert near(gr.project(S, ro, rd, **kw), I), kw
    assert near(gr.project_stats(S, ro, rd)[0], I)
    assert near(gr.project(S, ro, rd, precision="fp32"), gr.project(S, ro, rd, precision="fp32", waves_per_group=2))
    out = torch.full((m,), -1.0, device="cuda")
    cut = min(m, 64 * (1 + m // 200))
    gr.project_batched([S], [(0, ro, rd, 0, cut, out, 0), (0, ro, rd, cut, m - cut, out, cut)])
    assert near(out, I)
    rng = np.random.default_rng(6)
    off = rng.uniform(0.5, 1.5, m) * rng.choice([-1.0, 1.0], m)
    y = (ref["I_kappa"] + off * max(1e-3, float(ref["I_kappa"].mean()))).astype(np.float32)
    # (weights of the projection checked above: a pair on the cutoff, where either decision is right, moves its
    # ray's weight and with it every Gaussian on the ray)
    L, w = oracle.loss_weights("l2", I.cpu().numpy().astype(np.float64), y.astype(np.float64))
    want = oracle.grad(sc, o, d, w)
    idx = np.arange(n)
    for kw in (dict(), dict(hit_list_cap=64), dict(hit_list_cap=-1), dict(traversal=1), dict(persistent=2)):
        proj, loss = torch.empty(m, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        got = gr.project_backward(S, ro, rd, loss="l2", target=_dev(y), out_proj=proj, out_loss=loss, **kw)
        assert near(proj, I), kw
        assert abs(loss.item() - L) <= 1e-4 * L, kw
        assert_grad(gpu_grad_rows(got, idx), want, what=f"fused {kw}")
    w = sample_unit_weights(m, 3)
    want = oracle.grad(sc, o, d, w.astype(np.float64))
    for kw in (dict(), dict(waves_per_group=4), dict(persistent=2), dict(traversal=1)):
        assert_grad(gpu_grad_rows(gr.project_backward(S, ro, rd, _dev(w), **kw), idx), want, what=f"backward {kw}")
    want = oracle.grad_tof(sc, o, d, np.stack([w, -w, 0.5 * w]).astype(np.float64), 3, 40.0, 60.0)
    got = gr.project_tof_backward(S, ro, rd, _dev(np.stack([w, -w, np.float32(0.5) * w])), 3, sigma=40.0, bin_width=60.0)
    assert_grad(gpu_grad_rows(got, idx), want, what="tof backward")
    assert S.status_flags() == 0


# (leaf size: scenes of 20, 313 and 1 leaves): TOF forward of few packets, whose leaves are dealt out to the waves of
# a workgroup; one bin, bin counts on and past the rows exchanged at a time, and lines with nothing in reach
@pytest.mark.parametrize("n,leaf", [(320, 16), (313, 1), (60, 64)])
@pytest.mark.parametrize("bins", [0, 1, 15, 16, 17, 32])
def test_tof_forward_parts_against_oracle(gr, n, leaf, bins):
    import torch
    sc = sample_scene(n, seed=5 + n, radius=60.0, scale_range=(1.0, 9.0))
    rng = np.random.default_rng(n + bins)
    m = 64 * 12 + 17
    o = rng.uniform(-30, 30, (3, m)).astype(np.float32)
    d = rng.standard_normal((3, m)).astype(np.float32)
    d /= np.linalg.norm(d, axis=0)
    o[:, 64:128] = o[:, 64:65]
    d[:, 64:128] = d[:, 64:65] + np.float32(0.02) * d[:, 64:128]   # one coherent packet among scattered lines
    o[:, 200:210] += 500.0 * np.cross(d[:, 200:210], [0, 0, 1], axis=0)
    c = rng.uniform(-10, 10, m).astype(np.float32)
    att = rng.uniform(0.2, 1.0, m).astype(np.float32)
    sigma, width = 12.0, 9.0
    S = gr.Scene(*[_dev(a) for a in (sc.mean, sc.scale, sc.quat, sc.density)], leaf_size=leaf)
    kw = dict(center=_dev(c), atten=_dev(att))
    got = gr.project_tof(S, _dev(o), _dev(d), bins, sigma=sigma, bin_width=width, **kw)
    one = gr.project_tof(S, _dev(o), _dev(d), bins, sigma=sigma, bin_width=width, waves_per_group=2, **kw)
    ref = oracle.project_tof(sc, o, d, bins, sigma, width, center=c, atten=att)
    assert_bins(got.cpu().numpy(), ref, f"{n} Gaussians, {bins} bins")
    assert torch.allclose(got, one, rtol=LAST_BIT, atol=1e-37)
    assert S.status_flags() == 0


# (Gaussians, leaf size, scales, views): one coarse view whose packet has more candidates per wave than it lists
# (listed and own evaluations mixed), the most leaves that are shared by 16 and by fewer parts and one more
@pytest.mark.parametrize("n,leaf,views,nu", [(8192, 64, 1, 8), (128 * 4, 4, 1, 16), (128 * 4 + 1, 4, 1, 16),
                                             (1024, 2, 40, 40), (1026, 2, 40, 40), (2, 1, 1, 8)])
def test_shared_candidates_against_oracle(gr, n, leaf, views, nu):
    import torch
    sc = sample_scene(n, seed=3 + n, radius=60.0, scale_range=(1.0, 9.0))
    g = dict(kind="ct", cone=1, n_views=views, nu=nu, nv=nu, angle0=0.1, angle_range=5.0, dso=400.0, dsd=700.0,
             pitch_u=190.0 / nu, pitch_v=190.0 / nu, offset_u=0.0, offset_v=0.0, tile_u=8, tile_v=8)
    o, d = G.rays32(g)
    S = gr.Scene(*[_dev(a) for a in (sc.mean, sc.scale, sc.quat, sc.density)], leaf_size=leaf)
    I = gr.project(S, _dev(o), _dev(d))
    assert_forward(I.cpu().numpy(), oracle.project(sc, o, d), what=f"{n} {leaf}")
    for kw in (dict(), dict(traversal=1), dict(precision="fp32")):
        a = gr.project(S, _dev(o), _dev(d), **kw)
        assert a.cpu().numpy().tobytes() == gr.project(S, _dev(o), _dev(d), **kw).cpu().numpy().tobytes(), kw
        b = gr.project(S, _dev(o), _dev(d), waves_per_group=2, **kw)
        assert torch.allclose(a, b, rtol=LAST_BIT, atol=0.0), kw
    assert S.status_flags() == 0
