"""A launch of the serving loop looks at each waiting request once, also where
requests join it while it is prepared."""
import time

import pytest

import parity_util as U  # noqa: F401  (puts the package on the path)

pytestmark = pytest.mark.gpu


class Counting(dict):
    looks = 0

    def __getitem__(self, k):
        Counting.looks += 1
        return dict.__getitem__(self, k)


@pytest.mark.parametrize("moving", [False, True])
def test_each_request_is_looked_at_once(moving):
    from paper_1410_3219_amd import serve as S
    tpl = S.build_templates([400, 900], ["sod", "sod"], moving=moving)
    srv = S.Server(tpl, hbm_budget_bytes=1 << 30)
    waiting, steps = 300, 301
    srv.open_session(0, 0, steps)
    srv._admit()
    for rid in range(waiting):   # of one session: only the first can run
        srv.submit(rid, 0, 0.0)

    def poll():   # another session's first request joins
        srv.open_session(1, 1, 1)
        srv.submit(waiting, 1, 0.0)
        srv.poll = None
    srv.poll = poll
    srv.sessions = Counting(srv.sessions)
    Counting.looks = 0
    srv._launch()
    assert srv.launch_templates == [(0, 1)]
    # one for each request in the queue, one for the submission, and one for
    # each request that the launch takes
    assert Counting.looks <= waiting + 1 + 1 + 2, Counting.looks
    srv.sessions = dict(srv.sessions)
    t0 = time.perf_counter()
    while len(srv.done) < 2:
        srv._complete(lambda: time.perf_counter() - t0)
        assert time.perf_counter() - t0 < 30.0
    assert not srv.failed and sorted(r.rid for r in srv.done) == [0, waiting]
