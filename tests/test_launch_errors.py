"""A failed launch is reported, and nothing that reads its output is launched after it.

Where a call is several launches (adjoint splits and their sum, march classes, weight
gradient and its reductions), the runtime's last error after the final one says nothing
of the others: it is that of the last call.
"""
import pytest

import oracle
import tt_inputs as synth
from fake_hip import scenario
from geoms import tilted_angles


def _geometry(n, ell, n_rot, det, n_seg):
    inner, outer = tilted_angles(n_rot, (0.0, 27.0, 45.0), span_deg=360.0)
    return oracle.Geometry(n, ell, inner, outer, *det, n_seg, synth.lab_frame())


def projector_call(F, call, n, ell, n_rot, det, n_seg, batch):
    h = F.create(_geometry(n, ell, n_rot, det, n_seg))
    F.workspace(h, batch)
    sizes = F.sizes(h)
    c, y, out = F.buffer(4 * sizes[0]), F.buffer(4 * sizes[1]), F.buffer(4 * max(sizes[:2]))
    args = {"tt_adjoint": (h, y, out, 0.0, None), "tt_project": (h, c, out)}[call]
    rc, all_launches = F.launches(call, *args)
    assert rc == 0
    failed = []
    for i in range(len(all_launches)):
        F.rt.fake_fail_launch(i)
        rc, seen = F.launches(call, *args)
        failed.append((rc, len(seen)))
    return [name for name, *_ in all_launches], failed


def wgrad_call(F):
    n = F.ok("tt_conv3d_wgrad_work_bytes", 32, 32, 2, 16, 16, 16)
    b = F.buffer(1 << 20)
    args = (32, 32, b, b, 2, 16, 16, 16, F.buffer(n), n, F.buffer(4 * 27 * 1024), F.buffer(128), None)
    rc, all_launches = F.launches("tt_conv3d_wgrad", *args)
    assert rc == 0
    failed = []
    for i in range(len(all_launches)):
        F.rt.fake_fail_launch(i)
        rc, seen = F.launches("tt_conv3d_wgrad", *args)
        failed.append((rc, len(seen)))
    return [name for name, *_ in all_launches], failed


def _check(names, failed, kernels):
    assert all(any(k in name for name in names) for k in kernels), names
    for i, (rc, seen) in enumerate(failed):
        assert rc == -4 and seen == i, (names[i], rc, seen, i)


def test_adjoint_with_splits():
    _check(*scenario("test_launch_errors", "projector_call", "tt_adjoint", (8, 9, 10), 4, 43, (11, 12), 8, 1),
           ["k_fold", "k_backproject_win", "k_add_splits"])


@pytest.mark.parametrize("n_seg", [8, 16])
def test_march_in_several_launches(n_seg):
    names, failed = scenario("test_launch_errors", "projector_call", "tt_project", (8, 8, 8), 2, 60, (160, 160), n_seg,
                             180)
    _check(names, failed, ["k_map", "k_march_ring", "k_march"])
    assert len(names) >= 3


def test_weight_gradient():
    _check(*scenario("test_launch_errors", "wgrad_call"), ["k_wgrad", "k_wgrad_reduce", "k_bias_reduce"])
