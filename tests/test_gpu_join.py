"""Joined shells on the GPU.

On grids with n_phi = 2 n_theta a plan holds whole shells in the registers of
one workgroup for both passes: every plain shell that the theta pass filters
where a line has 48, 80, 96 or 128 points, and full rounds of one shell per
compute unit at 160, 192 and 256 points (a short last round takes two passes,
unless the other shells' rings fill the units).  The cases leave ragged
workgroups (two shells each at 80 points, four at 48), launches below and
above a round, a last round that is joined and one that is not, spread
shells, every kind and both parities.  Results match the oracle, equal the
two-pass filter to rounding, and in place and out of place are bitwise equal.
"""
import numpy as np
import pytest

import oracle
from paper_2305_01537_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-12        # against the oracle's direct transforms, as everywhere in these tests
TOL_TWO = 1e-14    # against the two-pass kernels: the same transforms, other contractions
EXP, GAUSS, SHARP, HYBRID = 0, 1, 2, 3


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def fields(shape, seed):
    """Smooth angular fields times a radial factor, plus noise."""
    F, R, T, P = shape
    rng = np.random.default_rng(seed)
    theta, phi = synth.theta_grid(T), synth.phi_grid(P)
    x = np.empty(shape)
    for f in range(F):
        a = synth.angular_sum(rng, 10, theta, phi, lambda l: 1.0 / (l + 1))
        x[f] = (1.0 + rng.random(R))[:, None, None] * a
    x += 1e-3 * rng.standard_normal(shape)
    parity = np.where(np.arange(F) % 2 == 0, 1, -1).astype(np.int32)
    x[parity < 0] *= np.sin(theta)[None, :, None]
    return x, parity


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


# shape (fields, shells, n_theta, n_phi), kinds, cal-L, rho (None: i + 1/2)
CASES = [
    ((1, 1, 24, 48), [EXP], 0.2, None),
    ((3, 3, 24, 48), [EXP, GAUSS, SHARP], 0.2, None),
    ((4, 11, 24, 48), [EXP, GAUSS, SHARP, HYBRID], 1.5, None),
    ((1, 1, 40, 80), [GAUSS], 0.2, None),
    ((3, 5, 40, 80), [EXP, GAUSS, SHARP], 0.2, None),
    ((4, 9, 40, 80), [EXP, GAUSS, SHARP, HYBRID], 3.0, None),
    ((4, 9, 48, 96), [EXP, GAUSS, SHARP, HYBRID], 3.0, None),
    ((4, 9, 64, 128), [EXP, GAUSS, SHARP, HYBRID], 4.0, None),
    ((3, 3, 80, 160), [EXP, GAUSS, SHARP], 0.5, None),       # a short round: two passes
    ((3, 60, 80, 160), [EXP, GAUSS, SHARP], 0.5, None),      # one round
    ((4, 70, 80, 160), [EXP, GAUSS, SHARP, HYBRID], 2.0, None),
    ((3, 60, 96, 192), [EXP, GAUSS, SHARP], 0.5, None),
    ((3, 91, 96, 192), [EXP, GAUSS, SHARP], 0.5, 1.0),       # a round and a short one
    ((2, 2, 128, 256), [EXP, SHARP], 3.0, None),
    ((3, 50, 128, 256), [EXP, GAUSS, SHARP], 1.0, None),     # one round
    ((3, 90, 128, 256), [EXP, GAUSS, SHARP], 0.5, 1.0),      # a round and a short one
    ((2, 400, 128, 256), [EXP, SHARP], 0.5, None),           # shells spread among the rings
]


@pytest.mark.parametrize("shape,kind,L,rho", CASES,
                         ids=["%dx%d-%dx%d-%s" % (*c[0], c[2]) for c in CASES])
def test_joined_shells(torch_gpu, shape, kind, L, rho):
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    F, R, T, P = shape
    x, parity = fields(shape, 311 + T)
    kind = np.array(kind, dtype=np.int32)
    hybrid = kind == HYBRID
    if hybrid.any():
        x[hybrid] += 3.0
        x[hybrid, R // 2, : T // 3, 1] = 0.0                 # a jump along theta
    rho = None if rho is None else np.full(R, rho)
    plan = Plan(R, T, P, F, parity=parity, L=L, rho=rho, kind=kind)
    st = plan.stats()
    print(f"[gpu] joined {shape} kinds {kind.tolist()} L {L}: theta shells {st['theta_shells_active']}",
          flush=True)
    for name, ref_fn in (("apply", oracle.forward), ("apply_adjoint", oracle.adjoint)):
        xd = torch.from_numpy(x).cuda()
        got = getattr(plan, name)(xd)
        assert torch.equal(xd, torch.from_numpy(x).cuda()), "the input of an out-of-place call"
        plan.set_fused(False)
        two = getattr(plan, name)(xd)
        plan.set_fused(True)
        assert torch.equal(getattr(plan, name)(xd, out=xd), got), "in place"
        got, two = got.cpu().numpy(), two.cpu().numpy()
        ref = ref_fn(x, parity=parity, L=np.full(F, L), rho=rho, kind=kind)
        for f in range(F):
            assert rel(got[f], ref[f]) <= TOL, (name, f, rel(got[f], ref[f]))
            assert rel(got[f], two[f]) <= TOL_TWO, (name, f, rel(got[f], two[f]))
    plan.close()


def test_joined_shells_pass_nonfinite_values_only_along_their_shell(torch_gpu):
    """An infinity stays inside its shell (all of it becomes non-finite, as the
    transforms spread it); every other shell of the launch is untouched by it."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    for T in (24, 40, 48, 64):
        shape = (2, 5, T, 2 * T)
        x, parity = fields(shape, 401)
        plan = Plan(5, T, 2 * T, 2, parity=parity, L=0.2, rho=np.ones(5))
        clean = plan.apply(torch.from_numpy(x).cuda())
        x[1, 2, 3, 4] = np.inf
        got = plan.apply(torch.from_numpy(x).cuda())
        bad = ~torch.isfinite(got)
        assert bad[1, 2].any()
        bad[1, 2] = False
        assert not bad.any()
        got[1, 2] = clean[1, 2]
        assert torch.equal(got, clean)
        plan.close()


def test_joined_shells_in_a_captured_graph(torch_gpu):
    """Forward and adjoint captured once, replayed with other work in between."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    shape = (2, 90, 80, 160)
    x, parity = fields(shape, 421)
    plan = Plan(90, 80, 160, 2, parity=parity, L=0.4)
    src = torch.from_numpy(x).cuda()
    eager = plan.apply_adjoint(plan.apply(src.clone()))
    buf = src.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        plan.apply(buf, out=buf)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.apply(buf, out=buf)
        plan.apply_adjoint(buf, out=buf)
    for k in range(3):
        buf.copy_(src)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(buf, eager), k
        _ = (src * 2.0).sum().item()
    plan.close()


@pytest.mark.parametrize("adjoint,inplace", [(False, True), (True, False)])
def test_joined_shells_in_a_batch(torch_gpu, adjoint, inplace):
    """A batch joins the shells of its plain n_phi = 2 n_theta patches, per line
    length over all patches: lengths with a round of shells (160: over two
    patches, 256: spread among the rings), with too few for one (192: two
    passes) and shorter ones, beside a patch with a hybrid field and one with
    another grid.  Every patch matches the oracle, and the call that allocates
    nothing gives the same bits."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Batch
    specs = [((2, 40, 80, 160), [EXP, GAUSS], 0.5), ((3, 41, 80, 160), [EXP, SHARP, EXP], 0.5),
             ((2, 400, 128, 256), [EXP, SHARP], 0.5), ((1, 7, 96, 192), [EXP], 0.5),
             ((3, 3, 40, 80), [EXP, GAUSS, SHARP], 1.5), ((1, 5, 24, 48), [SHARP], 1.5),
             ((2, 9, 64, 128), [EXP, HYBRID], 3.0), ((2, 9, 48, 96), [EXP, GAUSS], 3.0),
             ((2, 5, 32, 64), [EXP, EXP], 1.5), ((1, 9, 16, 32), [GAUSS], 0.5),
             ((2, 6, 32, 96), [EXP, GAUSS], 1.5), ((1, 3, 16, 32), [EXP], 50.0)]
    patches, data = [], []
    for i, (shape, kind, L) in enumerate(specs):
        x, parity = fields(shape, 500 + i)
        if HYBRID in kind:
            x += 3.0
        F, R, T, P = shape
        patches.append(dict(n_fields=F, n_r=R, n_theta=T, n_phi=P, parity=parity, L=L,
                            kind=np.array(kind, dtype=np.int32)))
        data.append(x)
    batch = Batch(patches)
    print(f"[gpu] batch of joined shells adjoint={adjoint} inplace={inplace}", flush=True)
    xs = [torch.from_numpy(x).cuda() for x in data]
    got = batch.apply(xs, outs=xs if inplace else None, adjoint=adjoint)
    again = [torch.from_numpy(x).cuda() for x in data]
    out2 = batch.apply_noalloc(again, outs=again if inplace else None, adjoint=adjoint)
    torch.cuda.synchronize()
    assert batch.status() == 0
    ref_fn = oracle.adjoint if adjoint else oracle.forward
    for p, x, g, g2 in zip(patches, data, got, out2):
        assert torch.equal(g, g2), p
        ref = ref_fn(x, parity=p["parity"], L=np.full(p["n_fields"], p["L"]), kind=p["kind"])
        assert rel(g.cpu().numpy(), ref) <= TOL, p
    batch.close()


@pytest.mark.parametrize("kind", [[EXP, SHARP, GAUSS, EXP, EXP, SHARP], [EXP, HYBRID, EXP, EXP, SHARP, EXP]])
def test_rings_straight_from_the_input_out_of_place(torch_gpu, kind):
    """Out of place, on a grid that is neither fused nor joined and where the rings
    of theta-idle shells move enough bytes, those rings go straight from the
    input to the output: bitwise the call in place, and the oracle's filter."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    shape = (6, 300, 32, 256)
    x, parity = fields(shape, 611)
    kind = np.array(kind, dtype=np.int32)
    x[kind == HYBRID] += 3.0
    L = np.full(6, 0.4)
    plan = Plan(300, 32, 256, 6, parity=parity, L=L, kind=kind)
    st = plan.stats()
    idle_rings = st["phi_rings_active"] - st["theta_shells_active"] * 32
    print(f"[gpu] direct rings {shape}: {idle_rings} rings of idle shells", flush=True)
    assert 32 * (idle_rings // 2) * 256 >= 96 << 20 and st["phi_rings_active"] < st["phi_rings_total"]
    xd = torch.from_numpy(x).cuda()
    got = plan.apply(xd)
    assert torch.equal(xd, torch.from_numpy(x).cuda())
    assert torch.equal(plan.apply(xd, out=xd), got)
    ref = oracle.forward(x, parity=parity, L=L, kind=kind)
    for f in range(6):
        assert rel(got[f].cpu().numpy(), ref[f]) <= TOL, f
    plan.close()


@pytest.mark.parametrize("shape,L,hybrid", [((24, 256, 64, 128), 1.0, False), ((24, 256, 64, 128), 1.0, True),
                                            ((24, 3600, 16, 32), 0.012, False), ((24, 1200, 32, 64), 0.18, True),
                                            ((8, 256, 96, 192), 1.0, False), ((10, 256, 96, 192), 1.0, True)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_two_passes_out_of_place_filter_every_ring(torch_gpu, shape, L, hybrid):
    """With fusing off, on grids that are fused or joined otherwise and where the
    rings of theta-idle shells move 96 MiB or more: the call out of place gives
    the bits of the call in place and the oracle's filter, and every byte of a
    hybrid field's decisions is written."""
    torch = torch_gpu
    from paper_2305_01537_amd.autograd import sph_filter
    from paper_2305_01537_amd.filter import Plan
    F, R, T, P = shape
    rng = np.random.default_rng(641)
    x = rng.standard_normal(shape)
    parity = np.where(np.arange(F) % 2 == 0, 1, -1).astype(np.int32)
    kind = np.where(np.arange(F) % 3 == 1, SHARP, EXP).astype(np.int32)
    if hybrid:
        kind[:2] = HYBRID
    plan = Plan(R, T, P, F, parity=parity, L=L, kind=kind)
    plan.set_fused(False)
    st = plan.stats()
    idle = st["phi_rings_active"] - st["theta_shells_active"] * T
    print(f"[gpu] two passes {shape} hybrid={hybrid}: {idle} rings of idle shells", flush=True)
    assert 32 * (idle // 2) * P >= 96 << 20
    xd = torch.from_numpy(x).cuda()
    want = plan.apply(xd.clone(), out=None)
    inplace = xd.clone()
    plan.apply(inplace, out=inplace)
    assert torch.equal(want, inplace)
    shells = [0, 1, R // 8, R // 4, R // 2, R - 1]
    rho = synth.uniform_rho(R)[shells]
    for f in (0, 1, F - 1):
        ref = oracle.forward(x[f:f + 1, shells], parity=parity[f:f + 1], L=np.full(1, L), rho=rho,
                             kind=kind[f:f + 1])
        got = want[f, shells].cpu().numpy()
        assert rel(got, ref[0]) <= TOL, (f, rel(got, ref[0]))
    if hybrid:
        dec = [torch.full(s, 255, dtype=torch.uint8, device="cuda") for s in ((F, R, P // 2), (F, R, T))]
        mine = [d.clone() for d in dec]
        plan.apply_ex(xd, theta_dec=dec[0], phi_dec=dec[1])
        y = xd.clone()
        plan.apply_ex(y, out=y, theta_dec=mine[0], phi_dec=mine[1])
        for a, b in zip(dec, mine):
            assert int(a[:2].max()) <= 1 and torch.equal(a, b)
        del a, b, y
        g = torch.from_numpy(rng.standard_normal(shape)).cuda()
        gref = plan.apply_ex(g, adjoint=True, theta_dec=dec[0], phi_dec=dec[1], replay=True)
        del dec, mine                       # their 255s are what the next empty buffers hold
        xd.requires_grad_(True)
        out = sph_filter(xd, plan)
        assert torch.equal(out.detach(), want)
        out.backward(g)
        assert torch.equal(xd.grad, gref)
    plan.close()


@pytest.mark.parametrize("shape,L", [((3, 40, 128, 256), 6.0), ((3, 30, 96, 192), 6.0), ((3, 20, 80, 160), 3.0),
                                     ((3, 12, 64, 96), 3.0), ((3, 150, 80, 160), 3.0), ((3, 256, 96, 192), 3.0),
                                     ((3, 142, 80, 160), 0.284)])
def test_few_plain_shells_beside_hybrid_ones_give_the_same_bits_everywhere(torch_gpu, shape, L):
    """Too few plain shells for a round beside hybrid shells in two passes, a full
    round of joined ones, a round of plain ones with more behind it (and a grid
    that is never joined): in place, out of place and with overlapped passes the
    bits are the same, and the oracle's filter."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    F, R, T, P = shape
    x, parity = fields(shape, 661 + T)
    x[0] += 3.0
    x[0, R // 2, : T // 3, 1] = 0.0
    kind = np.array([HYBRID, EXP, SHARP], dtype=np.int32)
    plan = Plan(R, T, P, F, parity=parity, L=L, kind=kind)
    st = plan.stats()
    assert 0 < st["theta_shells_active"] - R < 2 * R          # plain shells: some filtered, some idle
    print(f"[gpu] few plain shells {shape}", flush=True)
    xd = torch.from_numpy(x).cuda()
    for name, ref_fn in (("apply", oracle.forward), ("apply_adjoint", oracle.adjoint)):
        call = getattr(plan, name)
        got = call(xd)
        for overlap in (0, 2):
            plan.set_overlap(overlap)
            y = xd.clone()
            assert torch.equal(call(y, out=y), got), overlap
        plan.set_overlap(0)
        ref = ref_fn(x, parity=parity, L=np.full(F, L), kind=kind)
        for f in range(F):
            assert rel(got[f].cpu().numpy(), ref[f]) <= TOL, (name, f)
    plan.close()


@pytest.mark.parametrize("n_theta,n_r", [(16, 9), (24, 9), (32, 7), (40, 5), (48, 5), (64, 9), (80, 60), (96, 60),
                                         (128, 60)])
@pytest.mark.parametrize("adjoint,inplace", [(False, False), (True, True)])
def test_a_batch_of_one_line_length_is_joined(torch_gpu, n_theta, n_r, adjoint, inplace):
    """Two patches of one length, plain kinds, filtered and idle shells: joined
    (from a round of shells on at 160 points and more), against the oracle."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Batch
    shapes = [(3, n_r, n_theta, 2 * n_theta), (1, n_r + 2, n_theta, 2 * n_theta)]
    patches, data = [], []
    for i, shape in enumerate(shapes):
        x, parity = fields(shape, 700 + i + n_theta)
        F, R, T, P = shape
        rho = np.where(np.arange(R) % 5 == 4, 0.3 * T, 0.4)          # a fifth of the shells idle at cal-L = 2
        patches.append(dict(n_fields=F, n_r=R, n_theta=T, n_phi=P, parity=parity, L=2.0, rho=rho,
                            kind=np.array([EXP, SHARP, EXP][:F], dtype=np.int32)))
        data.append(x)
    batch = Batch(patches)
    print(f"[gpu] batch of one length {n_theta} adjoint={adjoint}", flush=True)
    xs = [torch.from_numpy(x).cuda() for x in data]
    got = batch.apply(xs, outs=xs if inplace else None, adjoint=adjoint)
    ref_fn = oracle.adjoint if adjoint else oracle.forward
    for p, x, g in zip(patches, data, got):
        ref = ref_fn(x, parity=p["parity"], L=np.full(p["n_fields"], 2.0), rho=p["rho"], kind=p["kind"])
        assert rel(g.cpu().numpy(), ref) <= TOL, p
    batch.close()


def test_small_unlike_patches_are_not_joined(torch_gpu):
    """A joined launch per length in a row would take longer than the two passes
    of all patches together: with joining on or off the same kernels run, and
    give the same bits."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Batch
    patches, data = [], []
    for i, T in enumerate((16, 24, 32, 40, 48, 64, 80, 96, 128)):
        shape = (3, 4, T, 2 * T)
        x, parity = fields(shape, 760 + i)
        patches.append(dict(n_fields=3, n_r=4, n_theta=T, n_phi=2 * T, parity=parity, L=3.0,
                            kind=np.array([EXP, GAUSS, SHARP], dtype=np.int32)))
        data.append(torch.from_numpy(x).cuda())
    batch = Batch(patches)
    print("[gpu] small unlike patches", flush=True)
    for adjoint in (False, True):
        on = batch.apply(data, adjoint=adjoint)
        batch.set_fused(False)
        off = batch.apply(data, adjoint=adjoint)
        batch.set_fused(True)
        for p, x, a, b in zip(patches, data, on, off):
            assert torch.equal(a, b), p
            ref = (oracle.adjoint if adjoint else oracle.forward)(
                x.cpu().numpy(), parity=p["parity"], L=np.full(3, 3.0), kind=p["kind"])
            assert rel(a.cpu().numpy(), ref) <= TOL, p
    batch.close()


@pytest.mark.parametrize("n_theta", [80, 96, 128])
def test_workgroups_that_loop_over_shells_keep_them_apart(torch_gpu, n_theta):
    """From eight shells per compute unit on, one workgroup per unit takes many
    shells with one LDS area: every shell equals the two-pass filter to rounding,
    and infinities stay inside their shells."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    R = 8 * torch.cuda.get_device_properties(0).multi_processor_count + 150
    shape = (1, R, n_theta, 2 * n_theta)
    plan = Plan(R, n_theta, 2 * n_theta, 1, parity=-1, L=0.2, rho=np.ones(R))
    print(f"[gpu] looping workgroups {shape}", flush=True)
    x = torch.randn(shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    hit = [0, 1, 255, 256, 257, 1000, R // 2, R - 151, R - 1]
    for name in ("apply", "apply_adjoint"):
        call = getattr(plan, name)
        got = call(x)
        plan.set_fused(False)
        two = call(x)
        plan.set_fused(True)
        size = two.abs().amax(dim=(2, 3))
        assert float(((got - two).abs().amax(dim=(2, 3)) / size).max()) <= TOL_TWO
        y = x.clone()
        y[0, hit, 3, 4] = float("inf")
        bad = call(y)
        keep = torch.ones(R, dtype=torch.bool, device="cuda")
        keep[hit] = False
        assert torch.equal(bad[0, keep], got[0, keep]), name
        assert not torch.isfinite(bad[0, hit]).flatten(1).all(dim=1).any(), name
        del got, two, y, bad
    plan.close()


@pytest.mark.parametrize("shape,L", [((2, 246, 80, 160), 0.896), ((4, 256, 128, 256), 3.0), ((3, 130, 96, 192), 2.0)])
def test_too_few_shells_to_join_out_of_place(torch_gpu, shape, L):
    """Too few filtered shells for a round, the rings of many idle ones: two
    passes, or with the rings straight from the input; the bits of the call in
    place, and the oracle's filter on sampled shells."""
    torch = torch_gpu
    from paper_2305_01537_amd.filter import Plan
    F, R, T, P = shape
    x = np.random.default_rng(811).standard_normal(shape)
    parity = np.where(np.arange(F) % 2 == 0, 1, -1).astype(np.int32)
    kind = np.where(np.arange(F) % 2 == 0, EXP, SHARP).astype(np.int32)
    plan = Plan(R, T, P, F, parity=parity, L=L, kind=kind)
    n = plan.stats()["theta_shells_active"]
    print(f"[gpu] too few shells to join {shape}: {n}", flush=True)
    assert 0 < 16 * n < 9 * torch.cuda.get_device_properties(0).multi_processor_count
    xd = torch.from_numpy(x).cuda()
    shells = [0, 1, R // 8, R // 4, R // 2, R - 1]
    for name, ref_fn in (("apply", oracle.forward), ("apply_adjoint", oracle.adjoint)):
        got = getattr(plan, name)(xd)
        y = xd.clone()
        assert torch.equal(getattr(plan, name)(y, out=y), got), name
        ref = ref_fn(x[:2, shells], parity=parity[:2], L=np.full(2, L), rho=synth.uniform_rho(R)[shells],
                     kind=kind[:2])
        for f in range(2):
            assert rel(got[f, shells].cpu().numpy(), ref[f]) <= TOL, (name, f)
    plan.close()
