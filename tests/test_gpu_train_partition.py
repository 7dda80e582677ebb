"""The training step over the edges of its launches: waves per workgroup and
partly filled workgroups, register- and slice-resident gradient tiles by layer
count, the workgroups' sums, the cell scan's two forms, and Adam in the
gradient kernels or in its own launch. Gradients against the FP64 oracle: within
1e-4 of the largest in FP32 (sums over thousands of points) and 3e-3 with FP16
network passes; one Adam update within 1e-6 of the oracle's for the same
gradients; dW the same bits in every call."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2112_01579_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "f16": 3e-3}


@pytest.fixture(scope="module")
def FV():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01579_amd import fvsrn
    fvsrn.lib()
    return fvsrn


def _rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


def _step(FV, spec, n, prec, key_times=None, seed=61):
    lat, w = I.net_params(spec, seed)
    gnet, onet = FV.Network(spec, lat, w, key_times), O.Net(spec, lat, w, key_times)
    rng = np.random.default_rng(seed + n)
    xyz = I.uniform_points(n, seed + 1, -0.99, 0.99)
    times = None
    d = O.eval_points(onet, xyz)
    if key_times is not None:
        times = rng.choice(np.array([-1.0, 0.0, 0.4, 1.0, 1.75, 9.0], np.float32), n)
        for t in np.unique(times):
            d[times == t] = O.eval_points(onet, xyz[times == t], float(t))
    # targets away from the prediction, so that sign(d - t) is the oracle's
    target = (d + rng.uniform(0.02, 0.3, n) * rng.choice([-1, 1], n)).astype(np.float32)
    dl_ref, dw_ref, loss_ref = O.train_grads(onet, xyz, target=target.astype(np.float64), times=times)
    cu = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
    out = []
    for _ in range(2):
        d_lat, d_w, loss = torch.empty_like(gnet.latent), torch.empty_like(gnet.weights), torch.zeros(1, device="cuda")
        FV.fvsrn_train_step(gnet, d_lat, d_w, cu(xyz), target=cu(target), times=cu(times), out_loss=loss, precision=prec)
        out.append((d_lat.cpu().numpy(), d_w.cpu().numpy(), loss.item()))
    assert np.array_equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]
    e_w, e_l = _rel(out[0][1], dw_ref), _rel(out[0][0], dl_ref)
    print("train c%d H%d R%d K%d n%d %s: dW %.3g dG %.3g loss %.3g" % (
        spec.c, spec.H, spec.R, spec.K, n, prec, e_w, e_l, abs(out[0][2] - loss_ref) / loss_ref), flush=True)
    assert e_w <= TOL[prec] and e_l <= TOL[prec]
    assert abs(out[0][2] - loss_ref) <= (1e-5 if prec == "f32" else 1e-3) * abs(loss_ref) + 1e-7


# 16-point chunks: 1 wave; one more point; 257 waves (65 workgroups of four, the
# last with one); 1022 (256 of four, the last with two); 1500 (250 of six); 2048
# and one chunk more (a ninth of a wave's chunks)
@pytest.mark.parametrize("n", [1, 16, 17, 16 * 257, 16 * 1021 + 5, 16 * 1500, 16 * 2048 + 16])
@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_train_wave_counts(FV, n, prec):
    _step(FV, I.NetSpec(R=8, F=8, L=4, c=32, H=3), n, prec)


@pytest.mark.parametrize("c,H", [(32, 1), (32, 2), (32, 4), (32, 8), (48, 1), (48, 2), (48, 8)])
@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_train_layer_counts(FV, c, H, prec):
    _step(FV, I.NetSpec(R=6, F=16, L=8, c=c, H=H), 3001, prec)


# 4096 cells (one block of the scan), 4913 (two), 64000 (16, each adding the
# counts before it) and 68921 (17, summed first)
@pytest.mark.parametrize("R", [2, 17, 18, 41, 42])
def test_train_cell_scan(FV, R):
    _step(FV, I.NetSpec(R=R, F=8, L=4, c=32, H=2), 2999, "f32")


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("n", [33, 5001])
def test_train_keyframes(FV, n, prec):
    _step(FV, I.NetSpec(R=5, F=16, L=8, c=32, H=2, K=3), n, prec, key_times=[0.0, 1.0, 2.5])


@pytest.mark.parametrize("K,R", [(1, 9), (1, 30), (3, 6)])
def test_train_adam_in_gradient_kernels(FV, K, R):
    """Two-pass latent gradient (K = 1, fits the slices) with Adam in its
    kernel, one-pass (K = 3) with Adam in a launch of its own; the weights'
    always in the kernel that writes their gradient. Nonzero moments, step 7."""
    spec = I.NetSpec(R=R, F=8, L=4, c=32, H=3, K=K)
    kt = [0.0, 1.0, 2.0] if K > 1 else None
    lat, w = I.net_params(spec, 71)
    gnet = FV.Network(spec, lat, w, kt)
    rng = np.random.default_rng(72)
    n = 4000
    xyz, target = I.uniform_points(n, 73), rng.uniform(0.0, 1.0, n).astype(np.float32)
    times = rng.uniform(0.0, 2.0, n).astype(np.float32) if K > 1 else None
    mom = {k: (rng.normal(0.0, 1e-4, s) if k[0] == "m" else rng.uniform(1e-9, 1e-8, s)).astype(np.float32)
           for k, s in (("m_latent", spec.n_latent), ("v_latent", spec.n_latent), ("m_weights", spec.n_weights),
                        ("v_weights", spec.n_weights))}
    opt = dict(lr_grid=1e-2, lr_mlp=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, step=7,
               **{k: torch.from_numpy(v).cuda() for k, v in mom.items()})
    d_lat, d_w = torch.empty_like(gnet.latent), torch.empty_like(gnet.weights)
    FV.fvsrn_train_step(gnet, d_lat, d_w, torch.from_numpy(xyz).cuda(), target=torch.from_numpy(target).cuda(), adam=opt,
                        times=None if times is None else torch.from_numpy(times).cuda())
    f = lambda x: float(np.float32(x))  # noqa: E731
    for p0, g, m, v, lr, p in ((lat.reshape(-1), d_lat, "m_latent", "v_latent", 1e-2, gnet.latent),
                                       (w, d_w, "m_weights", "v_weights", 1e-3, gnet.weights)):
        p64, m64, v64 = (a.astype(np.float64).copy() for a in (p0, mom[m], mom[v]))
        O.adam(p64, g.cpu().numpy().astype(np.float64), m64, v64, f(lr), f(0.9), f(0.999), f(1e-8), 7)
        assert np.abs(p.cpu().numpy() - p64).max() <= 1e-6
        assert np.abs(opt[m].cpu().numpy() - m64).max() <= 1e-6 * np.abs(m64).max()
        assert np.abs(opt[v].cpu().numpy() - v64).max() <= 1e-6 * np.abs(v64).max()


def _adam_step(FV, spec, kt, offset):
    """One step with moments in one flat buffer, `offset` floats into it."""
    lat, w = I.net_params(spec, 75)
    gnet = FV.Network(spec, lat, w, kt)
    rng = np.random.default_rng(76)
    n = 900
    xyz, target = I.uniform_points(n, 77), rng.uniform(0.0, 1.0, n).astype(np.float32)
    size = 2 * (spec.n_latent + spec.n_weights) + 4
    flat = torch.zeros(size, device="cuda")
    at, opt = offset, dict(lr_grid=1e-2, lr_mlp=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, step=3)
    for k in ("m_latent", "v_latent", "m_weights", "v_weights"):
        m = spec.n_latent if "latent" in k else spec.n_weights
        opt[k] = flat[at:at + m]
        opt[k].copy_(torch.from_numpy(rng.uniform(1e-9, 1e-8, m).astype(np.float32)))
        at += m
    d_lat, d_w = torch.empty_like(gnet.latent), torch.empty_like(gnet.weights)
    times = None if kt is None else torch.from_numpy(rng.uniform(0.0, 2.0, n).astype(np.float32)).cuda()
    FV.fvsrn_train_step(gnet, d_lat, d_w, torch.from_numpy(xyz).cuda(), target=torch.from_numpy(target).cuda(), adam=opt,
                        times=times)
    return [t.cpu().numpy() for t in (gnet.latent, gnet.weights, opt["m_latent"], opt["v_latent"], opt["m_weights"],
                                      opt["v_weights"], flat[:offset], flat[at:])]


@pytest.mark.parametrize("K", [1, 3])
@pytest.mark.parametrize("offset", [1, 2, 3])
def test_train_moments_at_any_float(FV, K, offset):
    """Moments that are views into a flat optimiser buffer, at no 16-byte boundary: the
    update of aligned ones (d_latent's sums may differ in their order, so to
    rounding), and nothing written beside them."""
    spec = I.NetSpec(R=7, F=8, L=4, c=32, H=2, K=K)
    kt = [0.0, 1.0, 2.0] if K > 1 else None
    a, b = _adam_step(FV, spec, kt, 0), _adam_step(FV, spec, kt, offset)
    for x, y in zip(a[:6], b[:6]):
        assert np.abs(x - y).max() <= 1e-6 * np.abs(x).max()
    assert (b[6] == 0.0).all() and (b[7] == 0.0).all()


@pytest.mark.parametrize("F,L,H,R,n", [(16, 8, 4, 32, 1 << 18), (16, 8, 6, 32, 1 << 20), (8, 4, 8, 64, 1 << 18)])
def test_train_two_pass_latent_gradient(FV, F, L, H, R, n):
    """Sparse single-keyframe grids sum per cell and corner first wherever the
    workspace holds those sums, in deep networks too, whose launches have fewer
    waves than the workspace has slices."""
    spec = I.NetSpec(R=R, F=F, L=L, c=32, H=H)
    lat, w = I.net_params(spec, 78)
    gnet = FV.Network(spec, lat, w)
    xyz, target = torch.rand(n, 3, device="cuda") * 2 - 1, torch.rand(n, device="cuda")
    d_lat, d_w = torch.empty_like(gnet.latent), torch.empty_like(gnet.weights)
    ws = torch.empty(FV.fvsrn_train_workspace_size(spec, n), dtype=torch.uint8, device="cuda")
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        FV.fvsrn_train_step(gnet, d_lat, d_w, xyz, target=target, workspace=ws)
        torch.cuda.synchronize()
    names = " ".join(e.key for e in prof.key_averages())
    assert "cell_partials_kernel" in names and "latent_grad_kernel" not in names
