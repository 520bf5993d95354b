"""Mixed batches whose processes do not all take the default FP64 kernels:
their common module holds graph bodies, and pair bodies beside them."""
import numpy as np
import pytest
import torch

from paper_2511_19456_amd import inputs
from parity import check_fp64, per_point_ref

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _segments(spec, prec):
    """Per (n, N, variant): the plan's segment, and its momenta and codes on the host."""
    from paper_2511_19456_amd.qedx import QedProcess
    segs, host = [], []
    for k, (n, N, var) in enumerate(spec):
        p = QedProcess(n, "per_point", prec, var)
        u, hel = inputs.rambo_inputs(500 + k, n, N, with_helicities=True)
        mom = p.rambo(torch.as_tensor(u, device=DEV), 6.0 + 3 * n)
        out = torch.full((N + 1,), -7.0, dtype=torch.float64, device=DEV)
        segs.append((p, mom, torch.as_tensor(hel.astype(np.int32), device=DEV), out[:N]))
        host.append((n, mom.cpu().numpy(), hel, out))
    return segs, host


@pytest.mark.parametrize("tile", [64, 256])
def test_fp32c_batch_without_the_fp64_pass(tile):
    """FP32C processes with the FP64 pass turned off.  A point whose diagram
    terms cancel by less than the pass's threshold (16, and the sum of the
    terms' magnitudes is at least the root of the sum of their squares) is one
    that the pass leaves alone, so FP32C's 1e-4 holds there."""
    from paper_2511_19456_amd.qedx import BatchPlan, make_variant
    off = make_variant(fixup=-1)
    segs, host = _segments([(3, 129, off), (6, 17, off), (1, 65, off), (5, 40, off), (2, 31, off), (4, 33, off)], "fp32c")
    plan = BatchPlan(segs, tile_points=tile)
    for rep in range(2):
        for h in host:
            h[3].fill_(-7.0)
        plan.launch()
        torch.cuda.synchronize()
        for n, mom, hel, out in host:
            ref, kap = per_point_ref(mom, n, hel)
            got = out.cpu().numpy()
            assert got[-1] == -7.0, n
            ok = kap <= 16.0
            assert ok.any() and np.abs(got[:-1][ok] / ref[ok] - 1.0).max() < 1e-4, (n, rep)


@pytest.mark.parametrize("tile", [64, 256, 0])
def test_default_and_explicit_shapes_in_one_batch(tile):
    """FP64: processes without a kernel shape (pair bodies) beside such with one
    (graph bodies: shared blocks, partition loops with and without the current
    cache, the distributive rewrite), each n in both forms; at 6 photons out the
    pair body alone fills the kernel's LDS."""
    from paper_2511_19456_amd.qedx import BatchPlan, make_variant
    explicit = {1: make_variant(block=256), 2: make_variant(rewrite=1, block=256), 3: make_variant(order=4),
                4: make_variant(order=1288), 5: make_variant(order=520), 6: make_variant(order=8)}
    spec = [(n, N, var) for n, N in ((1, 129), (2, 65), (3, 97), (4, 66), (5, 33), (6, 17)) for var in (None, explicit[n])]
    segs, host = _segments(spec, "fp64")
    plan = BatchPlan(segs, tile_points=tile)
    for rep in range(2):
        for h in host:
            h[3].fill_(-7.0)
        plan.launch()
        torch.cuda.synchronize()
        for (n, N, var), (_, mom, hel, out) in zip(spec, host):
            ref, kap = per_point_ref(mom, n, hel)
            got = out.cpu().numpy()
            assert got[-1] == -7.0, n
            check_fp64(got[:-1], ref, kap, f"n={n} {'explicit' if var else 'default'} shape, pass {rep}")


@pytest.mark.parametrize("var", [dict(order=8), dict(rewrite=1, block=256)])
def test_seven_photon_default_and_uncached_graph_body(var):
    """Both 7-photon bodies that would keep something in LDS."""
    from paper_2511_19456_amd.qedx import BatchPlan, make_variant
    segs, host = _segments([(6, 33, None), (6, 65, make_variant(**var))], "fp64")
    BatchPlan(segs, tile_points=64).launch()
    torch.cuda.synchronize()
    for n, mom, hel, out in host:
        ref, kap = per_point_ref(mom, n, hel)
        check_fp64(out.cpu().numpy()[:-1], ref, kap, f"n={n}")


@pytest.mark.parametrize("spec,tile", [([(1, 65)], 64), ([(6, 33), (2, 4097)], 64), ([(2, 300000), (5, 300000)], 64)])
def test_batch_info_counts_the_workgroups_started(spec, tile):
    """No more than four waves per workgroup have a tile to start with, and no
    more workgroups than four per compute unit are started."""
    from paper_2511_19456_amd.qedx import BatchPlan
    segs, host = _segments([(n, N, None) for n, N in spec], "fp64")
    info = BatchPlan(segs, tile_points=tile).info()
    tiles = sum(-(-N // 32) for n, N in spec)     # two lanes per point
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    assert info["tiles"] == tiles
    assert 1 <= info["grid"] <= min(-(-tiles // 4) + len(spec) - 1, 4 * ncu)
    if tiles > 16 * ncu:                          # a full round of every kernel: one and two workgroups per unit
        assert info["grid"] == 3 * ncu


@pytest.mark.parametrize("tile", [64, 1024])
def test_default_fp64_batch_has_the_eval_kernels_bits(tile):
    """Plans of processes without a kernel shape: their module and the eval
    kernels form FMAs alike."""
    from paper_2511_19456_amd.qedx import BatchPlan, make_variant
    spec = [(n, N, None) for n, N in ((6, 65), (5, 257), (4, 1030), (3, 999), (2, 4097), (1, 333))]
    spec += [(6, 33, make_variant(rewrite=1)), (3, 130, make_variant(rewrite=1))]
    segs, host = _segments(spec, "fp64")
    BatchPlan(segs, tile_points=tile).launch()
    torch.cuda.synchronize()
    for (p, mom, hel, out), (n, N, _) in zip(segs, spec):
        assert torch.equal(out, p.eval(mom, hel)), (n, N)
