"""The kernels with one current per photon subset, at the sizes where their
tiling can go wrong, against the oracle.

Per point (two lanes per point, 128 points per workgroup; five- and six-photon
kernels loop over the points with one workgroup per compute unit): single
points, the edges of a wave and of a workgroup, a ragged second round of the
loop.  Tolerances are those of tests/parity.py, derived from the oracle's own
cancellation.
"""
import numpy as np
import pytest
import torch

from paper_2511_19456_amd import inputs
from parity import check_fp64, per_point_ref

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n_in,n", [(1, 1), (1, 2), (1, 3), (1, 4), (1, 5), (1, 6), (3, 1), (5, 1), (2, 3)])
def test_per_point_tile_edges(n_in, n):
    """Every size on a prefix of the same points: equal results wherever a
    point lands in the grid, and the points at the edges against the oracle."""
    from paper_2511_19456_amd.qedx import QedProcess
    P = n + n_in
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    top = 128 * ncu + 129 if P in (5, 6) else 1000   # the loop's second round
    if n_in == 1:
        u, hel = inputs.rambo_inputs(70 + n, n, top, with_helicities=True)
        mom = QedProcess(n, "per_point").rambo(torch.as_tensor(u, device=DEV), 6.0 + 3 * n)
    elif n == 1:
        m, hel = inputs.crossed_inputs(70 + n_in, n_in, top, with_helicities=True)
        mom = torch.as_tensor(m, device=DEV)
    else:  # one outgoing photon of e- gamma -> e- 4 gamma crossed into the initial state
        u, _ = inputs.rambo_inputs(75, 4, top)
        m = QedProcess(4, "per_point").rambo(torch.as_tensor(u, device=DEV), 9.0).view(7, 4, top)
        mom = torch.cat([m[:2], -m[3:4], m[2:3], m[4:]]).reshape(28, top).contiguous()
        hel = inputs.rng_for(76).integers(0, 1 << 7, size=top).astype(np.uint32)
    p = QedProcess(n, "per_point", n_in=n_in)
    hd = torch.as_tensor(hel.astype(np.int32), device=DEV)
    full = p.eval(mom, hd)
    for N in (1, 2, 31, 32, 33, 127, 128, 129, top - 1):
        out = torch.full((N + 1,), -7.0, dtype=torch.float64, device=DEV)
        p.eval(mom[:, :N].contiguous(), hd[:N].contiguous(), out=out[:N])
        assert torch.equal(out[:N], full[:N]) and out[N].item() == -7.0, N
    idx = np.unique([0, 1, 31, 32, 63, 127, 128, top // 2, max(0, top - 129), top - 2, top - 1])
    ref, kap = per_point_ref(mom[:, idx].cpu().numpy(), n, hel[idx], n_in=n_in)
    check_fp64(full[idx].cpu().numpy(), ref, kap, f"{n_in} -> {n}")


def test_per_point_every_configuration_sums_to_the_helicity_sum():
    """All 2^(n+3) configurations of a point, one per lane pair, against the
    oracle's helicity sum (spin and polarisation codes of every particle)."""
    from oracle import qed_oracle as O
    from paper_2511_19456_amd.qedx import QedProcess
    n, k = 3, 5
    u, _ = inputs.rambo_inputs(77, n, k)
    mom = O.momenta_soa_from_uniforms(u, 10.0, n)
    hel = np.tile(np.arange(64, dtype=np.int32), k)
    mm = torch.as_tensor(np.repeat(mom.numpy(), 64, axis=1), device=DEV)
    got = QedProcess(n, "per_point").eval(mm, torch.as_tensor(hel, device=DEV)).view(k, 64).sum(1).cpu().numpy()
    ref = O.m2(mom, n, "sum").numpy()
    assert np.abs(got / ref - 1).max() < 1e-10


@pytest.mark.parametrize("n_in,n", [(1, 1), (1, 2), (1, 3), (1, 4), (2, 2), (4, 1)])
def test_helicity_sum_tile_edges(n_in, n):
    from oracle import qed_oracle as O
    from paper_2511_19456_amd.qedx import QedProcess
    top = 151
    if n_in == 1:
        u, _ = inputs.rambo_inputs(80 + n, n, top)
        mom = O.momenta_soa_from_uniforms(u, 5.0 + 3 * n, n).numpy()
    elif n == 1:
        mom, _ = inputs.crossed_inputs(80 + n_in, n_in, top)
    else:
        u, _ = inputs.rambo_inputs(85, 3, top)
        m = O.momenta_from_uniforms(u, 9.0, 3)
        mom = O.points_to_soa(torch.cat([m[:, :2], -m[:, 3:4], m[:, 2:3], m[:, 4:]], dim=1)).numpy()
    p = QedProcess(n, "sum", n_in=n_in)
    md = torch.as_tensor(mom, device=DEV)
    full = p.eval(md)
    ref = O.m2(mom, n, "sum", n_in=n_in).numpy()
    assert np.abs(full.cpu().numpy() / ref - 1).max() < 1e-10
    w = 64 // p.info()["lanes_per_point"]
    sizes = {1, 2, w - 1, w, w + 1} | {w * k for k in range(2, 10)} | {w * 7 + 1, w * 8 + 1, top - 1}
    for N in sorted(s for s in sizes if 0 < s < top):
        out = torch.full((N + 1,), -7.0, dtype=torch.float64, device=DEV)
        p.eval(md[:, :N].contiguous(), out=out[:N])
        assert torch.equal(out[:N], full[:N]) and out[N].item() == -7.0, N


@pytest.mark.parametrize("n,sqrt_s", [(1, 4.0), (2, 6.0), (3, 10.0), (4, 15.0)])
def test_gradient_tile_edges(n, sqrt_s):
    """Prefixes of one point set: the same values and gradients whatever the
    grouping, and the edge points against the oracle's reverse mode."""
    from oracle import qed_oracle as O
    from paper_2511_19456_amd.qedx import QedProcess
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    top = 300 if n == 4 else 8 * ncu * 16 + 37     # two groups per wave and a ragged end, at least
    u, _ = inputs.rambo_inputs(90 + n, n, top)
    ud = torch.as_tensor(u, device=DEV)
    p = QedProcess(n, "sum")
    val, g = p.eval_grad(ud, sqrt_s)
    assert bool(torch.isfinite(val).all()) and bool(torch.isfinite(g).all())
    for N in (1, 2, 3, 4, 5, 7, 8, 9, 31, 33, 65, 131, top - 1):
        v1 = torch.full((N + 1,), -7.0, dtype=torch.float64, device=DEV)
        g1 = torch.full((4 * (n + 1) * N + 1,), -7.0, dtype=torch.float64, device=DEV)
        p.eval_grad(ud[:, :N].contiguous(), sqrt_s, out=(v1[:N], g1[:-1].view(4 * (n + 1), N)))
        assert torch.equal(v1[:N], val[:N]) and v1[N].item() == -7.0, N
        assert torch.equal(g1[:-1].view(4 * (n + 1), N), g[:, :N]) and g1[-1].item() == -7.0, N
    idx = np.unique([0, 1, 3, 4, 7, 8, 15, 16, 31, 63, 64, top // 2, top - 2, top - 1])
    v_o, g_o = O.logm2_and_grad(u[:, idx], sqrt_s, n)
    assert np.abs(val[idx].cpu().numpy() - v_o.numpy()).max() < 1e-10 * max(1.0, np.abs(v_o.numpy()).max())
    err = np.linalg.norm(g[:, idx].cpu().numpy() - g_o.numpy(), axis=0) / np.linalg.norm(g_o.numpy(), axis=0)
    assert err.max() < 1e-10


@pytest.mark.parametrize("tile", [64, 256, 4096, 0])
@pytest.mark.parametrize("big", [False, True])
def test_batch_tile_ranges(tile, big):
    """Mixed batches cut into per-wave tile ranges, below and above the size
    from which each class of processes has its own kernel: empty, single-point
    and ragged segments, several of one process, classes without a segment.
    Every point against the per-process kernel (same code per point, so the
    rounding of one reordered sum at most) and none written past its end."""
    from paper_2511_19456_amd.qedx import BatchPlan, QedProcess
    spec = [(3, 65), (6, 33), (1, 1), (5, 0), (2, 4097), (6, 1), (4, 130), (3, 31), (1, 777)]
    if big:
        ncu = torch.cuda.get_device_properties(0).multi_processor_count
        spec += [(2, 900 * ncu + 5), (1, 200 * ncu + 31), (6, 4 * ncu + 3)]   # no 4 or 5 photon bulk
    procs, segs, ends, refs = {}, [], [], []
    for k, (n, N) in enumerate(spec):
        p = procs.setdefault(n, QedProcess(n, "per_point"))
        u, hel = inputs.rambo_inputs(400 + k, n, N, with_helicities=True)
        mom = p.rambo(torch.as_tensor(u, device=DEV), 6.0 + 3 * n)
        h = torch.as_tensor(hel.astype(np.int32), device=DEV)
        buf = torch.full((N + 1,), -7.0, dtype=torch.float64, device=DEV)
        ends.append(buf)
        segs.append((p, mom, h, buf[:N]))
        refs.append(p.eval(mom, h) if N else buf[:0].clone())
    plan = BatchPlan(segs, tile_points=tile)
    for rep in range(2):
        for b in ends:
            b.fill_(-7.0)
        plan.launch()
        torch.cuda.synchronize()
        for (n, N), b, r in zip(spec, ends, refs):
            assert b[N].item() == -7.0, (n, N)
            assert N == 0 or ((b[:N] - r).abs() <= 1e-13 * r.abs()).all(), (n, N, rep)
