"""FP32 sine networks on the FP16 matrix cores (every operand a pair of FP16
values): densities and images against the FP64 oracle where the split can go
wrong -- weights and latents far from 1, the smallest and largest layer counts,
odd widths, partial waves, every grid type at both channel counts, keyframes,
and four outputs.

Tolerance: the densities of the FP32 path are within 1e-5 of the oracle. A
weight scaled by 2^k scales the FP32 rounding of a pre-activation and so the
error of everything behind it, by at most 2^k per hidden layer it applies to;
those tests scale one layer and allow 2^k times the bound."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2112_01579_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def FV():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01579_amd import fvsrn
    fvsrn.lib()
    return fvsrn


def _nets(FV, spec, lat, w, grid="f32", key_times=None):
    gd = {"f32": FV.F32, "f16": FV.F16, "u8": FV.U8}[grid]
    gnet = FV.Network(spec, lat, w, key_times=key_times, grid_dtype=gd)
    if grid == "u8":
        codes, dq = zip(*[O.quantize_grid(lat[k].reshape(-1, spec.F), spec.F) for k in range(spec.K)])
        return gnet, O.Net(spec, None, w, key_times, codes=np.stack(codes), dequant=np.stack(dq))
    if grid == "f16":
        lat = lat.astype(np.float16).astype(np.float64)
    return gnet, O.Net(spec, lat, w, key_times)


def _density_error(FV, spec, lat, w, n, grid="f32", key_times=None, time=0.0, seed=5):
    gnet, onet = _nets(FV, spec, lat, w, grid, key_times)
    xyz = I.uniform_points(n, seed, -1.05, 1.05)  # a few points outside the domain
    d = FV.fvsrn_eval_points(gnet, torch.from_numpy(xyz).cuda(), time).cpu().numpy()
    return float(np.abs(d - O.eval_points(onet, xyz, time)).max())


@pytest.mark.parametrize("c,F,L,H", [(32, 8, 4, 1), (32, 16, 8, 8), (48, 16, 4, 1), (48, 8, 8, 5), (64, 16, 8, 2),
                                     (64, 8, 4, 8)])
@pytest.mark.parametrize("n", [1, 63, 65, 1000])
def test_split_shapes(FV, c, F, L, H, n):
    spec = I.NetSpec(R=5, F=F, L=L, c=c, H=H)
    lat, w = I.net_params(spec, 21 + c + H)
    err = _density_error(FV, spec, lat, w, n)
    print("split c%d F%d L%d H%d n%d err %.3g" % (c, F, L, H, n, err), flush=True)
    assert err <= TOL


@pytest.mark.parametrize("F,L", [(8, 4), (16, 8)])
@pytest.mark.parametrize("grid", ["f32", "f16", "u8"])
@pytest.mark.parametrize("K", [1, 3])
def test_split_grids(FV, F, L, grid, K):
    spec = I.NetSpec(R=7, F=F, L=L, c=32, H=3, K=K)
    lat, w = I.net_params(spec, 31 + F)
    kt = [0.0, 1.0, 3.0] if K > 1 else None
    err = _density_error(FV, spec, lat, w, 777, grid, kt, 1.5 if K > 1 else 0.0)
    print("split %s F%d K%d err %.3g" % (grid, F, K, err), flush=True)
    assert err <= TOL


@pytest.mark.parametrize("layer", [0, 1, 2])
@pytest.mark.parametrize("log2", [-40, -12, 3, 5])
def test_split_weight_ranges(FV, layer, log2):
    """One layer's weights times 2^log2: far below and above FP16's own range
    of hi and lo parts without the row scale."""
    spec = I.NetSpec(R=6, F=8, L=4, c=32, H=3)
    lat, w = I.net_params(spec, 41)
    at = 0
    for i, (o, k) in enumerate(spec.layer_shapes()):
        if i == layer:
            w[at:at + o * k] *= np.float32(2.0 ** log2)
        at += o * k + o
    err = _density_error(FV, spec, lat, w, 900)
    print("split layer %d x 2^%d err %.3g" % (layer, log2, err), flush=True)
    assert err <= TOL * max(1.0, 2.0 ** log2)


def test_split_rows_of_unlike_scale(FV):
    """Rows of one matrix 2^30 apart: each row has a scale of its own."""
    spec = I.NetSpec(R=6, F=8, L=4, c=32, H=3)
    lat, w = I.net_params(spec, 42)
    at = spec.layer_shapes()[0][0] * (spec.layer_shapes()[0][1] + 1)
    rows = w[at:at + 32 * 32].reshape(32, 32)
    rows[::2] *= np.float32(2.0 ** -30)
    rows[1::4] *= np.float32(2.0)
    err = _density_error(FV, spec, lat, w, 900)
    print("split unlike rows err %.3g" % err, flush=True)
    assert err <= 2 * TOL


@pytest.mark.parametrize("log2", [-60, 17])
def test_split_latent_ranges(FV, log2):
    """Latents outside FP16's range, with layer 0's latent weights scaled back:
    both stay in FP32."""
    spec = I.NetSpec(R=6, F=16, L=4, c=32, H=2)
    lat, w = I.net_params(spec, 43)
    lat = (lat * np.float32(2.0 ** log2)).astype(np.float32)
    o, k = spec.layer_shapes()[0]
    w[:o * k].reshape(o, k)[:, 3:3 + spec.F] *= np.float32(2.0 ** -log2)
    err = _density_error(FV, spec, lat, w, 900)
    print("split latents x 2^%d err %.3g" % (log2, err), flush=True)
    assert err <= TOL


def test_split_predicted_gradient(FV):
    spec = I.NetSpec(R=9, F=16, L=8, c=48, H=4, outputs=4)
    lat, w = I.net_params(spec, 44)
    gnet, onet = _nets(FV, spec, lat, w)
    xyz = I.uniform_points(1001, 6)
    d, g = FV.fvsrn_pred_grad_points(gnet, torch.from_numpy(xyz).cuda())
    dr, gr = (np.array(v) for v in zip(*(O.density_grad(onet, p, mode="pred") for p in xyz.astype(np.float64))))
    err = float(np.abs(d.cpu().numpy() - dr).max())
    gerr = float(np.abs(g.cpu().numpy() - gr).max() / np.abs(gr).max())
    print("split predicted err %.3g grad rel %.3g" % (err, gerr), flush=True)
    assert err <= TOL and gerr <= TOL


@pytest.mark.parametrize("c,F,L,H", [(32, 8, 4, 1), (32, 16, 8, 4), (48, 16, 8, 2), (48, 8, 4, 3), (48, 16, 8, 3),
                                     (48, 8, 4, 4), (32, 16, 8, 5)])
@pytest.mark.parametrize("grid", ["f32", "f16", "u8"])
def test_split_adjoint(FV, c, F, L, H, grid):
    """Adjoint gradients at the layer counts on both sides of the split's limits
    (registers: H = 4, LDS: c = 48), between keyframes, partial waves, a few
    points outside the domain; the bound of the FP32 gradients, 1e-5 of the
    largest."""
    spec = I.NetSpec(R=6, F=F, L=L, c=c, H=H, K=2)
    lat, w = I.net_params(spec, 51 + c + H)
    gnet, onet = _nets(FV, spec, lat, w, grid, [0.0, 2.0])
    xyz = I.uniform_points(205, 8, -1.05, 1.05)
    dr, gr = (np.array(v) for v in zip(*(O.density_grad(onet, p, 0.5, mode="rev") for p in xyz.astype(np.float64))))
    for n in (1, 63, 205):
        d, g = FV.fvsrn_grad_points(gnet, torch.from_numpy(xyz[:n]).cuda(), 0.5, "f32", mode="adjoint")
        err = float(np.abs(d.cpu().numpy() - dr[:n]).max())
        gerr = float(np.abs(g.cpu().numpy() - gr[:n]).max() / max(1.0, np.abs(gr).max()))
        print("split adjoint c%d F%d H%d %s n%d err %.3g grad rel %.3g" % (c, F, H, grid, n, err, gerr), flush=True)
        assert err <= TOL and gerr <= TOL


@pytest.mark.parametrize("layer,log2", [(0, -30), (1, -30), (2, 3), (3, -40)])
def test_split_adjoint_weight_ranges(FV, layer, log2):
    """One layer's weights times 2^log2: deltas far below FP16's range. Relative to
    the largest gradient; a layer scaled up by 2^k raises the bound by 2^k."""
    spec = I.NetSpec(R=6, F=8, L=4, c=32, H=3)
    lat, w = I.net_params(spec, 41)
    at = 0
    for i, (o, k) in enumerate(spec.layer_shapes()):
        if i == layer:
            w[at:at + o * k] *= np.float32(2.0 ** log2)
        at += o * k + o
    gnet, onet = _nets(FV, spec, lat, w)
    xyz = I.uniform_points(300, 9)
    _, g = FV.fvsrn_grad_points(gnet, torch.from_numpy(xyz).cuda(), 0.0, "f32", mode="adjoint")
    gr = np.array([O.density_grad(onet, p, mode="rev")[1] for p in xyz.astype(np.float64)])
    gerr = float(np.abs(g.cpu().numpy() - gr).max() / np.abs(gr).max())
    print("split adjoint layer %d x 2^%d grad rel %.3g" % (layer, log2, gerr), flush=True)
    assert gerr <= TOL * max(1.0, 2.0 ** log2)


@pytest.mark.parametrize("c,F,L,H,outputs", [(32, 16, 8, 4, 1), (32, 8, 4, 1, 1), (48, 16, 8, 4, 1), (48, 8, 4, 2, 4),
                                             (32, 16, 8, 5, 1), (32, 8, 8, 3, 1), (64, 16, 8, 2, 1)])
@pytest.mark.parametrize("n", [16 * 256, 16 * 256 * 9 + 1, 70001])
def test_forward_mode_gradients_at_many_points(FV, c, F, L, H, outputs, n):
    """FP32 forward-mode gradients on both sides of the point count beyond which
    the adjoint evaluates them, with and without an adjoint kernel for the shape:
    the FP32 gradients' bound at points spread over the call, the last one
    among them."""
    spec = I.NetSpec(R=6, F=F, L=L, c=c, H=H, outputs=outputs)
    lat, w = I.net_params(spec, 61 + c + H)
    gnet, onet = _nets(FV, spec, lat, w)
    xyz = I.uniform_points(n, 10, -1.02, 1.02)
    d, g = (v.cpu().numpy() for v in FV.fvsrn_grad_points(gnet, torch.from_numpy(xyz).cuda(), 0.0, "f32"))
    at = np.linspace(0, n - 1, 97).astype(np.int64)
    dr, gr = (np.array(v) for v in zip(*(O.density_grad(onet, p, 0.0) for p in xyz[at].astype(np.float64))))
    err, gerr = float(np.abs(d[at] - dr).max()), float(np.abs(g[at] - gr).max() / max(1.0, np.abs(gr).max()))
    print("forward c%d F%d H%d n%d err %.3g grad rel %.3g" % (c, F, H, n, err, gerr), flush=True)
    assert err <= TOL and gerr <= TOL and np.isfinite(g).all()


def test_split_largest_network(FV):
    """c = 64, F = 16, L = 8, H = 8: one wave per CU beside its 153 KB of fragments, for
    points and for a view."""
    spec = I.NetSpec(R=5, F=16, L=8, c=64, H=8)
    lat, w = I.net_params(spec, 93)
    gnet, onet = _nets(FV, spec, lat, w)
    assert _density_error(FV, spec, lat, w, 20001) <= TOL
    cams, m = I.orbit_cameras(2, 9, 7), I.March(step=1.0 / 20)
    img = FV.fvsrn_render(gnet, I.ramp_tf(), cams, m).cpu().numpy()
    ref, _ = O.render(O.Field(net=onet), I.ramp_tf(), cams, m)
    assert float(np.abs(img - ref).max()) <= TOL
