"""FP16 and BF16 point evaluation, where lanes of a wave share the loads of
their samples' vertices: densities against the FP64 oracle, and each point's
density independent (bit for bit) of the points beside it in the batch.

Tolerances: those of the FP16 and BF16 networks elsewhere, 3e-3 and 3e-2."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2112_01579_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = {"f16": 3e-3, "bf16": 3e-2}


@pytest.fixture(scope="module")
def FV():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_01579_amd import fvsrn
    fvsrn.lib()
    return fvsrn


@pytest.mark.parametrize("F,L", [(8, 4), (16, 8)])
@pytest.mark.parametrize("K", [1, 2])
@pytest.mark.parametrize("grid", ["f32", "f16", "u8"])
@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_points_share_loads(FV, prec, grid, K, F, L):
    spec = I.NetSpec(R=7, F=F, L=L, c=32, H=2, K=K)
    lat, w = I.net_params(spec, 71 + F)
    kt = [0.0, 2.0] if K == 2 else None
    t = 0.75 if K == 2 else 0.0
    gnet = FV.Network(spec, lat, w, key_times=kt, grid_dtype={"f32": FV.F32, "f16": FV.F16, "u8": FV.U8}[grid])
    if grid == "u8":
        codes, dq = zip(*[O.quantize_grid(lat[k].reshape(-1, F), F) for k in range(K)])
        onet = O.Net(spec, None, w, kt, codes=np.stack(codes), dequant=np.stack(dq))
    else:
        onet = O.Net(spec, lat.astype(np.float16).astype(np.float64) if grid == "f16" else lat, w, kt)
    xyz = I.uniform_points(131, 12, -1.05, 1.05)
    x = torch.from_numpy(xyz).cuda()
    d = FV.fvsrn_eval_points(gnet, x, t, prec)
    err = float(np.abs(d.cpu().numpy() - O.eval_points(onet, xyz, t)).max())
    print("shared loads %s %s K%d F%d err %.3g" % (prec, grid, K, F, err), flush=True)
    assert err <= TOL[prec]
    for n in (1, 2, 3, 66):
        assert torch.equal(FV.fvsrn_eval_points(gnet, x[:n].contiguous(), t, prec), d[:n])
    back = torch.flip(x, [0]).contiguous()
    assert torch.equal(torch.flip(FV.fvsrn_eval_points(gnet, back, t, prec), [0]), d)
