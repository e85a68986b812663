"""sdp_time_stages on the one-pass products with B: the members of a cluster
exchange their sums through words tagged with the number of the pass, so a
launch under the number of the one before it finds them there and waits for
nobody.  Every timed launch has to be a pass of its own."""
import pytest

import sdpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algorithm", ["primal", "dual", "hsde"])
def test_every_launch_is_a_pass(sdp, gpu, algorithm):
    inst = sdpgen.banded_instance(600, 15, 301, seed=5)
    n = 7
    with sdp.Solver([inst], algorithm=algorithm, tol=0.0, max_iter=1000) as S:
        start = S.affine_plan()
        assert start["workgroups"] > 0 and start["part_bytes"] > 0
        S.step(5)
        steps = S.affine_plan()["passes"]
        assert steps == start["passes"] + 5
        ms = S.time_stages(n)
        # stage 4's launches alone, and with those of stage 1
        assert S.affine_plan()["passes"] == steps + 2 * n
        assert all(v >= 0.0 for v in ms.values()) and ms["A_v"] > 0.0 and ms["AT_y"] > 0.0


def test_two_passes(sdp, gpu):
    with sdp.Solver([sdpgen.block_arrow_instance(4, 5, 3, 15, seed=1)], tol=0.0) as S:
        S.step(3)
        S.time_stages(4)
        assert S.affine_plan() == dict(workgroups=0, part_bytes=0, passes=0)
