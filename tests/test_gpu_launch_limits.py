"""z segments up to the number of planes: two segment-end rows each, together
beyond a grid's second extent (65535).  A state uniform along z gives the planes
of a short lattice, to the rounding of sums that the segments order differently
(FP64 1e-12; FP32 with the surrogate, whose acceptance threshold is 1e-6 of T,
1e-5 of the largest population)."""
import numpy as np
import pytest

from paper_2510_14712_amd import inputs

pytestmark = pytest.mark.gpu

ST = inputs.states()
RHOC, TC = ST["critical"]["rho"], ST["critical"]["T"]


@pytest.mark.parametrize("storage,eos,nseg", [("f64", "vdw", 65535), ("f64", "vdw", 32768), ("f32", "mlp", 40000)])
def test_segments_up_to_the_planes(storage, eos, nseg):
    from paper_2510_14712_amd import lbm
    lbm.load()
    nx, ny, nz = 8, 4, 65535
    print(f"case {storage} {eos} {nseg} segments", flush=True)
    rho, u, T = inputs.random_state(2, (nx, ny), 35, RHOC, 1.1 * TC, drho=0.03, du=0.05, dT=0.02, white=0.005)
    u = np.concatenate([u.reshape(2, -1), np.zeros((1, nx * ny))])
    net = None
    if eos == "mlp":
        box = ST["shock_drop_3d"]["mlp_box"]
        net = lbm.mlp_train([*box["rho"], *box["T"]], 16384, 9, 2, 4096, 3e-3, inputs.mlp_params(9).astype(np.float32))
    out = []
    for n, segs in ((8, 1), (nz, nseg)):
        tall = [np.ascontiguousarray(np.broadcast_to(a[:, None], (a.shape[0], n, nx * ny))).reshape(-1)
                for a in (rho.reshape(1, -1), u, T.reshape(1, -1))]
        with lbm.Lattice(3, (nx, ny, n), storage=storage, eos=eos, mlp_tol=1e-6, zsegments=segs,
                         **inputs.physics(ST)) as lat:
            assert lat.fused
            if net is not None:
                lat.mlp_set(net[0], net[1])
            lat.init(*tall).step(3)
            lat.synchronize()
            out.append([p.view(27, n, nx * ny).cpu() for p in lat.get_populations()])
    tol = 1e-12 if storage == "f64" else 1e-5
    for a, b in zip(*out):
        assert float((b - a[:, :1]).abs().max()) <= tol * float(a.abs().max())
