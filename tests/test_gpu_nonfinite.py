"""Infinities where they have no effect in FP32 arithmetic on one sample after the
other: behind the sample that ends a ray, in a weight of the output layer, in the
gradient of one point of a cell."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2112_01579_amd import inputs as I

pytestmark = pytest.mark.gpu

# transparent at density 0, opaque within one step of 1/40 from density 0.01 on
HARD_TF = I.TF(points=((0.0, 0.2, 0.4, 0.9, 0.0), (0.01, 0.2, 0.4, 0.9, 1.0), (1.0, 1.0, 0.6, 0.2, 1.0)),
               opacity_scale=500.0)


@pytest.fixture(scope="module")
def FV():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01579_amd import fvsrn
    fvsrn.lib()
    return fvsrn


@pytest.mark.parametrize("w,h", [(33, 21), (200, 150)])
def test_dense_infinity_behind_the_surface(FV, w, h):
    """A volume that rises to 3e38 behind an opaque slab, Phong: the infinite gradient
    belongs to samples that no ray composites."""
    vol = np.ones((48, 40, 44), np.float32)  # the camera looks along -z: z = +1 is in front
    hidden = vol.copy()
    hidden[:40] = 3e38
    m = I.March(step=1.0 / 40, ert_eps=1e-3, phong=True)
    a, b = (FV.fvsrn_render_dense(torch.from_numpy(v).cuda(), HARD_TF, [I.ortho_camera(w, h)], m).cpu().numpy()
            for v in (vol, hidden))
    assert np.isfinite(a).all() and a[..., 3].max() > 0.99
    assert np.array_equal(a, b)


@pytest.mark.parametrize("w,h", [(32, 24), (90, 60)])
def test_render_infinity_behind_the_surface(FV, w, h):
    """The same for the network: latents of 3e38 in every other vertex layer from 0.27
    units behind the face on give finite densities and infinite gradients."""
    spec = I.NET_SMALL
    lat, weights = I.net_params(spec, 51)
    far = lat.copy().reshape(spec.K, spec.R, spec.R, spec.R, spec.F)
    far[:, :spec.R - 3:2, ..., 0] = 3e38
    m = I.March(step=1.0 / 40, ert_eps=1e-3, phong=True, grad_mode=3)
    a, b = (FV.fvsrn_render(FV.Network(spec, v.reshape(lat.shape), weights), HARD_TF, [I.ortho_camera(w, h)], m,
                            "f32").cpu().numpy() for v in (lat, far))
    assert np.isfinite(a).all() and a[..., 3].max() > 0.99
    assert np.array_equal(a, b)
