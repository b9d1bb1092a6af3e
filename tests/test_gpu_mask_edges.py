"""Sharp filters whose ring cutoffs lie a few units of the last place from an
integer, on shells that the theta pass leaves alone (2 rho cal-L >= n_theta,
so only rings near the poles are filtered).  Which modes such a ring keeps is
decided by the FP64 value of its cutoff, 2 rho sin(theta_j) cal-L, as in the
oracle: a mode kept or dropped wrongly is an error of the order of the field.
"""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 1e-12        # against the oracle's direct transforms, as everywhere in these tests
SHARP = 2


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def edge_rhos(n_theta, L):
    """Radii of theta-idle shells that give ring 0 a cutoff 0 to 3 units of the
    last place below or above an integer from 2 to 8."""
    s = math.sin(0.5 * math.pi / n_theta)
    rhos, below = [], 0
    for q in range(2, 9):
        rho = np.nextafter(q / (2.0 * s * L), 0.0)
        for _ in range(8):
            rho = np.nextafter(rho, 0.0)
        for _ in range(24):
            rho = np.nextafter(rho, np.inf)
            c = 2.0 * rho * s * L
            if c >= 2.0 and abs(c - q) <= 3 * np.spacing(float(q)) and 2.0 * rho * L >= n_theta:
                rhos.append(float(rho))
                below += c < q
    assert below >= 6 and len(rhos) > below
    return np.array(sorted(set(rhos)))


def sharp_patch(n_theta, L, seed):
    rho = edge_rhos(n_theta, L)
    shape = (2, len(rho), n_theta, 2 * n_theta)
    x = np.random.default_rng(seed).standard_normal(shape)
    x[:, :, n_theta // 2:] *= 1e-3           # mirror rings of unlike size: a leak between them shows
    return dict(n_fields=2, n_r=len(rho), n_theta=n_theta, n_phi=2 * n_theta,
                parity=np.array([1, -1], dtype=np.int32), L=L, rho=rho,
                kind=np.full(2, SHARP, dtype=np.int32)), x


def reference(p, x, adjoint):
    ref_fn = oracle.adjoint if adjoint else oracle.forward
    return ref_fn(x, parity=p["parity"], L=np.full(2, p["L"]), rho=p["rho"], kind=p["kind"])


def rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


@pytest.mark.parametrize("n_theta", [16, 24, 32, 40, 48, 64, 80, 96, 128])
@pytest.mark.parametrize("adjoint", [False, True])
def test_sharp_rings_at_the_edge_of_a_mode(torch_gpu, n_theta, adjoint):
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    p, x = sharp_patch(n_theta, 3.0, 700 + n_theta)
    plan = Plan(**p)
    assert plan.stats()["theta_shells_active"] == 0
    # a shell that the theta pass filters, so that a plan joins or fuses
    q = dict(p, n_r=p["n_r"] + 1, rho=np.append(p["rho"], 0.5))
    z = np.concatenate([x, x[:, :1]], axis=1)
    for prm, data in ((p, x), (q, z)):
        with Plan(**prm) as pl:
            print(f"[gpu] sharp edges {data.shape} adjoint={adjoint}", flush=True)
            xd = torch.from_numpy(data).cuda()
            got = (pl.apply_adjoint if adjoint else pl.apply)(xd, out=xd).cpu().numpy()
        ref = reference(prm, data, adjoint)
        for f in range(2):
            for i in range(data.shape[1]):
                for half in (slice(0, n_theta // 2), slice(n_theta // 2, n_theta)):
                    err = rel(got[f, i, half], ref[f, i, half])
                    assert err <= 1e3 * TOL, (f, i, err)         # the halves differ in size by 1e3
                assert rel(got[f, i], ref[f, i]) <= TOL, (f, i)
    plan.close()


@pytest.mark.parametrize("adjoint", [False, True])
def test_sharp_rings_at_the_edge_of_a_mode_in_a_batch(torch_gpu, adjoint):
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Batch
    patches, data = zip(*[sharp_patch(T, 3.0, 800 + T) for T in (16, 24, 32, 40, 48, 64)])
    # one filtered shell each, so that the patch's line length is joined
    for p in patches:
        p["n_r"] += 1
        p["rho"] = np.append(p["rho"], 0.5)
    data = [np.concatenate([x, x[:, :1]], axis=1) for x in data]
    batch = Batch(list(patches))
    print(f"[gpu] sharp edges in a batch adjoint={adjoint}", flush=True)
    xs = [torch.from_numpy(x).cuda() for x in data]
    for p, x, g in zip(patches, data, batch.apply(xs, outs=xs, adjoint=adjoint)):
        assert rel(g.cpu().numpy(), reference(p, x, adjoint)) <= TOL, p["n_theta"]
    batch.close()
