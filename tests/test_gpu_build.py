"""The acceleration structure at the sizes where its build changes form: the
one-launch sort's last size and the first past it, sort tiles, leaves that do
not fill a workgroup, two levels of the hierarchy above the one-workgroup top,
equal codes and invalid Gaussians among them. Both traversals against the FP64
oracle, after a build and after a refit of moved Gaussians."""
import numpy as np
import pytest

import oracle
from paper_2602_01057_amd.inputs import Scene, sample_scene
from parity import assert_forward

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _check(gr, S, sc, o, d, what):
    ref = oracle.project(sc, o, d)
    assert (ref["hits"] > 0).sum() > o.shape[1] // 4
    for traversal in (1, 2):
        assert_forward(gr.project(S, _dev(o), _dev(d), traversal=traversal).cpu().numpy(), ref,
                       what=f"{what} traversal {traversal}")
    assert S.status_flags() == 0


@pytest.mark.parametrize("n,leaf", [(1, 64), (64, 64), (65, 64), (127, 1), (129, 2), (1023, 48), (1025, 7), (4096, 64),
                                    (4096, 1), (4097, 64), (5119, 33), (12_288, 64), (12_289, 5), (70_001, 1),
                                    (140_000, 64)])
def test_build_and_refit_against_oracle(gr, n, leaf):
    rng = np.random.default_rng(n + leaf)
    hi = 9.0 * max(1.0, n / 500) ** -0.2
    sc = sample_scene(n, seed=n, radius=50.0, scale_range=(hi / 6, hi))
    if n == 1:
        sc = Scene(0 * sc.mean, 0 * sc.scale + 40.0, sc.quat, sc.density)
    mean, scale, quat, dens = (a.copy() for a in (sc.mean, sc.scale, sc.quat, sc.density))
    if n > 100:
        mean[:, n // 3:n // 3 + 70] = mean[:, :1]        # a leaf and more of equal codes
        bad = rng.choice(n, 9, replace=False)
        scale[0, bad[:3]] = 0.0
        quat[:, bad[3:6]] = 0.0
        mean[1, bad[6:]] = np.nan
    P = [_dev(a) for a in (mean, scale, quat, dens)]
    S = gr.Scene(*P, leaf_size=leaf)
    m = 200
    o = rng.uniform(-25, 25, (3, m)).astype(np.float32)
    d = rng.standard_normal((3, m)).astype(np.float32)
    n_bad = 9 if n > 100 else 0
    assert S.invalid_count() == n_bad
    _check(gr, S, Scene(mean, scale, quat, dens), o, d, "build")
    # moved, resized, one more invalid; then a build over the same workspace
    mean2 = mean + rng.normal(0, 1.5, mean.shape).astype(np.float32)
    scale2 = scale * rng.uniform(0.9, 1.2, scale.shape).astype(np.float32)
    if n > 100:
        scale2[2, 5] = -1.0
    for t, a in zip(P, (mean2, scale2, quat, dens)):
        t.copy_(_dev(a))
    bad2 = int((~np.isfinite(mean2).all(0) | ~(scale2 > 0).all(0) | ~(np.abs(quat).sum(0) > 0)).sum())
    S.refit()
    assert S.invalid_count() == bad2
    _check(gr, S, Scene(mean2, scale2, quat, dens), o, d, "refit")
    S.build()
    assert S.invalid_count() == bad2
    _check(gr, S, Scene(mean2, scale2, quat, dens), o, d, "rebuild")


def test_all_invalid(gr):
    import torch
    n = 300
    sc = sample_scene(n, seed=1, radius=40.0)
    S = gr.Scene(_dev(sc.mean), _dev(-sc.scale), _dev(sc.quat), _dev(sc.density))
    o, d = np.zeros((3, 70), np.float32), np.ones((3, 70), np.float32)
    assert S.invalid_count() == n
    for traversal in (1, 2):
        assert float(gr.project(S, _dev(o), _dev(d), traversal=traversal).abs().max()) == 0.0
    g = gr.project_backward(S, _dev(o), _dev(d), torch.ones(70, device="cuda"))
    assert all(float(v.abs().max()) == 0.0 for v in g.values())
