"""Renders whose waves take several consecutive segments of a ray per step
(small launches): images and sample counts against the FP64 oracle at each
number of segments, shading mode and march, with and without early ray
termination.

The number of segments follows from the chord's length in steps: a small
launch takes 2, 4, 8 and 16 of them from a longest chord of 8, 16, 32 and 64
segments on (central differences, eight lanes per sample, at most 8)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
from paper_2112_01579_amd import inputs as I

pytestmark = pytest.mark.gpu

FP32_TOL, PHONG32_TOL, FP16_TOL = 1e-5, 2e-5, 3e-3
PER_UNIT = [2, 3, 6, 16, 40]  # longest chord 6.9, 10.4, 20.8, 55, 139 segments: 1, 2, 4, 8, 16 per step


@pytest.fixture(scope="module")
def FV():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01579_amd import fvsrn
    fvsrn.lib()
    return fvsrn


def _nets(FV, outputs=1):
    spec = dataclasses.replace(I.NET_SMALL, outputs=outputs)
    lat, w = I.net_params(spec, 51)
    return FV.Network(spec, lat, w), O.Net(spec, lat, w)


def _render(FV, gnet, cams, m, prec):
    stats = torch.zeros(3, dtype=torch.int64, device="cuda")
    img = FV.fvsrn_render(gnet, I.ramp_tf(), cams, m, prec, stats=stats).cpu().numpy()
    return img, stats.cpu().numpy()


# a ragged perspective view whose rays graze the box's edges, next to one from inside it
def _cams():
    inside = I.Camera(ortho=False, eye=(0.3, -0.2, 0.1), target=(1.0, 0.4, -0.3), up=(0.0, 1.0, 0.0), width=37,
                      height=23, fov_y_deg=80.0)
    return [I.orbit_cameras(3, 37, 23)[1], inside]


@pytest.mark.parametrize("per_unit", PER_UNIT)
@pytest.mark.parametrize("prec,tol", [("f32", FP32_TOL), ("f16", FP16_TOL)])
def test_segments_unshaded(FV, per_unit, prec, tol):
    gnet, onet = _nets(FV)
    m = I.March(step=1.0 / per_unit)
    img, stats = _render(FV, gnet, _cams(), m, prec)
    ref, ns = O.render(O.Field(net=onet), I.ramp_tf(), _cams(), m)
    err = float(np.abs(img - ref).max())
    print("segments %s 1/%d err %.3g" % (prec, per_unit, err), flush=True)
    assert err <= tol
    assert stats[0] == ns and stats[2] >= ns and stats[2] % 64 == 0


@pytest.mark.parametrize("fixed", [1, 9, 17, 33, 129])
def test_segments_fixed_steps(FV, fixed):
    gnet, onet = _nets(FV)
    m = I.March(step=0.0, fixed_steps=fixed)
    cams = [I.ortho_camera(19, 11)]
    img, stats = _render(FV, gnet, cams, m, "f32")
    ref, ns = O.render(O.Field(net=onet), I.ramp_tf(), cams, m)
    assert float(np.abs(img - ref).max()) <= FP32_TOL
    assert stats[0] == ns == stats[1] * fixed and stats[1] == 11 * 11  # the view is wider than the box


@pytest.mark.parametrize("per_unit", PER_UNIT)
@pytest.mark.parametrize("eps", [0.02, 0.3])
def test_segments_termination(FV, per_unit, eps):
    """A ray ends behind the sample that took T below eps, wherever that is in
    its step: every pixel matches the oracle's at eps, or, where T comes
    within 1e-4 of it, at one of the neighbouring thresholds."""
    gnet, onet = _nets(FV)
    cams = _cams()
    img, stats = _render(FV, gnet, cams, I.March(step=1.0 / per_unit, ert_eps=eps), "f32")
    refs = [O.render(O.Field(net=onet), I.ramp_tf(), cams, I.March(step=1.0 / per_unit, ert_eps=e))
            for e in (eps, eps * (1 - 1e-4), eps * (1 + 1e-4))]
    err = np.min([np.abs(img - r).max(-1) for r, _ in refs], axis=0)
    print("segments ERT %g 1/%d err %.3g" % (eps, per_unit, err.max()), flush=True)
    assert float(err.max()) <= FP32_TOL
    counts = [n for _, n in refs]
    assert min(counts) <= stats[0] <= max(counts)


@pytest.mark.parametrize("per_unit", PER_UNIT)
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_segments_shaded(FV, per_unit, mode):
    gnet, onet = _nets(FV, 4 if mode == 2 else 1)
    m = I.March(step=1.0 / per_unit, phong=True, grad_mode=mode, fd_step=1.0 / 32.0 if mode == 1 else 0.0)
    img, stats = _render(FV, gnet, _cams(), m, "f32")
    ref, _ = O.render(O.Field(net=onet), I.ramp_tf(), _cams(), m)
    _, ns = O.render(O.Field(net=onet), I.ramp_tf(), _cams(), I.March(step=1.0 / per_unit))
    err = float(np.abs(img - ref).max())
    print("segments shaded %d 1/%d err %.3g" % (mode, per_unit, err), flush=True)
    assert err <= PHONG32_TOL
    assert stats[0] == ns


def test_segments_rays_that_miss(FV):
    """Tiles with no ray in the box, and with one."""
    gnet, onet = _nets(FV)
    cam = I.Camera(ortho=False, eye=(0.0, 0.0, 3.0), target=(0.0, 2.2, 0.0), up=(0.0, 1.0, 0.0), width=41, height=40)
    m = I.March(step=1.0 / 40)
    img, stats = _render(FV, gnet, [cam], m, "f32")
    ref, ns = O.render(O.Field(net=onet), I.ramp_tf(), [cam], m)
    assert float(np.abs(img - ref).max()) <= FP32_TOL and stats[0] == ns
    assert 0 < stats[1] < 41 * 40


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("mode", [None, 3])
def test_segments_of_rays_that_end_at_once(FV, prec, mode):
    """A transfer function of one extinction ends every ray at its fourth sample
    (exp(-500 / 256 * 4) < 1e-3 < exp(-500 / 256 * 3)), whatever the densities. At over
    a tile per wave the launch may not spend several times as many slots on it."""
    gnet, _ = _nets(FV)
    tf = I.TF(points=((0.0, 0.9, 0.5, 0.1, 1.0), (1.0, 1.0, 0.6, 0.2, 1.0)), opacity_scale=500.0)
    m = I.March(step=1.0 / 256, ert_eps=1e-3, phong=mode is not None, grad_mode=mode or 0)
    stats = torch.zeros(3, dtype=torch.int64, device="cuda")
    img = FV.fvsrn_render(gnet, tf, [I.ortho_camera(640, 640)], m, prec, stats=stats).cpu().numpy()
    n, rays, slots = stats.cpu().numpy()
    print("solid %s mode %s: %d samples of %d rays in %d slots" % (prec, mode, n, rays, slots), flush=True)
    assert rays == 640 * 640 and n == 4 * rays and slots <= 1.5 * n
    assert float(np.abs(img[..., 3] - (1.0 - np.exp(-500.0 / 256 * 4))).max()) <= 1e-5


# Networks whose forward-mode Phong has a kernel of its own (four lanes per sample): the
# FP16 passes, FP32 above four layers, and a shape without an adjoint.
FORWARD = [("f16", I.NET_SMALL, 1e-2), ("f32", dataclasses.replace(I.NET_SMALL, H=5), PHONG32_TOL),
           ("f32", I.NetSpec(R=9, F=16, L=4, c=32, H=2), PHONG32_TOL)]


def _forward_net(FV, spec):
    lat, w = I.net_params(spec, 52)
    return FV.Network(spec, lat, w), O.Net(spec, lat, w)


@pytest.mark.parametrize("prec,spec,tol", FORWARD)
def test_segments_forward_mode(FV, prec, spec, tol):
    """1, 2, 4, 8 and 16 segments of a ray per step, 16 samples per wave step: the
    slots issued are multiples of 16, and not of the other kernels' 64."""
    gnet, onet = _forward_net(FV, spec)
    odd = 0
    for per_unit in PER_UNIT:
        m = I.March(step=1.0 / per_unit, phong=True)
        img, stats = _render(FV, gnet, _cams(), m, prec)
        ref, _ = O.render(O.Field(net=onet), I.ramp_tf(), _cams(), m)
        _, ns = O.render(O.Field(net=onet), I.ramp_tf(), _cams(), I.March(step=1.0 / per_unit))
        err = float(np.abs(img - ref).max())
        print("segments forward %s H%d 1/%d err %.3g" % (prec, spec.H, per_unit, err), flush=True)
        assert err <= tol and stats[0] == ns and stats[2] % 16 == 0
        odd += stats[2] % 64 != 0
    assert odd > 0


@pytest.mark.parametrize("prec,spec,tol", FORWARD)
@pytest.mark.parametrize("per_unit", [3, 6, 40])
def test_segments_forward_mode_termination(FV, prec, spec, tol, per_unit):
    gnet, onet = _forward_net(FV, spec)
    cams, eps = _cams(), 0.3
    img, stats = _render(FV, gnet, cams, I.March(step=1.0 / per_unit, ert_eps=eps, phong=True), prec)
    near = 1e-4 if prec == "f32" else 1e-2  # of T around eps, by the densities' error
    refs = [O.render(O.Field(net=onet), I.ramp_tf(), cams, I.March(step=1.0 / per_unit, ert_eps=e, phong=True))
            for e in (eps, eps * (1 - near), eps * (1 + near))]
    err = np.min([np.abs(img - r).max(-1) for r, _ in refs], axis=0)
    counts = [O.render(O.Field(net=onet), I.ramp_tf(), cams, I.March(step=1.0 / per_unit, ert_eps=e))[1]
              for e in (eps * (1 + near), eps * (1 - near))]
    print("segments forward ERT %s H%d 1/%d err %.3g" % (prec, spec.H, per_unit, err.max()), flush=True)
    assert float(err.max()) <= tol and min(counts) <= stats[0] <= max(counts)
