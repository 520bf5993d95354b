"""qed_eval over more points than one launch's threads."""
import ctypes

import pytest
import torch

from paper_2511_19456_amd import _lib, inputs

DEV = "cuda:0"


def _ranges(N, lanes, block, most):
    L, v = _lib.lib(), [ctypes.c_int64() for _ in range(3)]
    out, i = [], 0
    while not out or i < out[0][0]:
        assert L.qed_launch_range(N, lanes, block, most, i, *[ctypes.byref(x) for x in v]) == 0
        out.append(tuple(x.value for x in v))
        i += 1
    assert L.qed_launch_range(N, lanes, block, most, i, *[ctypes.byref(x) for x in v]) == _lib.QED_ERR_INVALID_ARG
    return out


@pytest.mark.parametrize("lanes,block", [(32, 64), (8, 64), (4, 64), (2, 256), (2, 64), (1, 64)])
@pytest.mark.parametrize("most", [64 * 4, 1000, 4097, 2 ** 32 - 1])
def test_ranges_cover_every_point_within_the_limit(lanes, block, most):
    tile, full = block // lanes, most // block * (block // lanes)
    sizes = {1, full - 1, full, full + 1, 2 * full, 2 * full + 1, 3 * full - tile, 5 * full + 3, 17 * full + tile - 1}
    for N in sorted(s for s in sizes if s > 0):
        if most < block:
            continue
        r = _ranges(N, lanes, block, most)
        end = 0
        for count, first, points in r:
            assert count == len(r) == -(-N // full) and 0 <= first <= end and first + points <= N
            end = max(end, first + points)
            threads = -(-points * lanes // block) * block
            assert threads <= most
            # in one launch the kernel's own bound is N; in several no thread is past the launch's points
            assert count == 1 or threads == points * lanes
        assert end == N


@pytest.mark.gpu
def test_helicity_sum_over_two_launches():
    """5 photons, 32 lanes per point: 2^27 points are one launch's threads."""
    from paper_2511_19456_amd.qedx import QedProcess
    n, N, K = 4, (1 << 27) + 77, 4099
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 48 GB of device memory")
    p = QedProcess(n, "sum")
    info = p.info()
    assert len(_ranges(N, info["lanes_per_point"], info["block"], 2 ** 32 - 1)) == 2
    u, _ = inputs.rambo_inputs(91, n, K)
    base = p.rambo(torch.as_tensor(u, device=DEV), 15.0)
    ref = p.eval(base)
    reps = -(-N // K)
    mom = torch.empty(28, N, dtype=torch.float64, device=DEV)
    for r in range(28):
        mom[r] = base[r].repeat(reps)[:N]
    out = torch.full((N + 1,), -7.0, dtype=torch.float64, device=DEV)
    p.eval(mom, out=out[:N])
    assert torch.equal(out[:N], ref.repeat(reps)[:N]) and out[N].item() == -7.0
