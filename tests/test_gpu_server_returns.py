"""The serving pool where a call ends early or a walker leaves between sweeps:
the walkers that stay give the numbers they give alone, bit for bit."""
import time

import pytest

from gpu_util import require_gpu
from paper_1708_00744_amd import dsu, inputs

pytestmark = pytest.mark.gpu

L, K = 10.0, 16


def request(rid, n, spins=1, sweeps=3, arrival_s=0.0, sigma=0.2):
    pos = inputs.positions(17, rid, spins * n, L).reshape(spins, n, 3)
    return {"request_id": rid, "n": n, "spins": spins, "seed": 17, "sigma": sigma, "sweeps": sweeps,
            "arrival_s": arrival_s, "positions": pos}


def add(server, r):
    return server.add(r["request_id"], r["n"], r["spins"], r["seed"], r["sigma"], r["sweeps"], r["positions"])


def pool(prec, recompute_every=0):
    return dsu.Server(K, precision=prec, box_l=L, budget_bytes=1 << 30, recompute_every=recompute_every)


def alone(prec, r, sweeps, recompute_every=0):
    with pool(prec, recompute_every) as s:
        slot = add(s, r)
        for _ in range(sweeps):
            s.step()
        return s.result(slot, remove=True)


def numbers(result):
    return {q: result[q] for q in ("request_id", "status", "sweeps_done", "logdet", "sign", "accepted")}


@pytest.mark.parametrize("prec", [dsu.FP64, dsu.FP32_MIXED])
@pytest.mark.parametrize("bad", [{"spins": 3}, {"sweeps": -1}])
def test_refused_run_leaves_walkers_with_their_inverses(prec, bad):
    """A request that is refused ends the run; those placed before it stay
    resident, are swept by later steps and leave or are joined as any other."""
    require_gpu()
    reqs = [request(1, 96), request(2, 96, spins=2), request(3, 64)]
    with pool(prec) as s:
        with pytest.raises(dsu.DsuError) as ex:
            s.run(reqs + [request(4, 80, **bad)])
        assert ex.value.code == dsu.EINVAL
        assert s.usage()[1] == 3
        s.step()
        gone = s.result(0, remove=True)
        late = request(5, 96)
        slot = add(s, late)
        s.step()
        rest = [s.result(q, remove=True) for q in (1, 2, slot)]
        assert s.usage() == (0, 0)
    assert numbers(gone) == numbers(alone(prec, reqs[0], 1))
    for got, r, sweeps in zip(rest, reqs[1:] + [late], (2, 2, 1)):
        assert numbers(got) == numbers(alone(prec, r, sweeps))


@pytest.mark.parametrize("prec", [dsu.FP64, dsu.FP32_MIXED])
def test_recompute_where_another_walker_leaves(prec):
    """Recomputes every three sweeps; the walker first in the list leaves at the
    sweep after which the others are due.  The inverse a recompute gives differs
    from the updated one by rounding, so the numbers after further sweeps tell
    whether it took place, and on which walker."""
    require_gpu()
    reqs = [request(11, 96, spins=2, sweeps=3), request(12, 96, sweeps=7), request(13, 96, spins=2, sweeps=7)]
    with pool(prec, recompute_every=3) as s:
        results, _ = s.run(reqs)
        assert s.usage() == (0, 0)
    for got, r in zip(results, reqs):
        assert numbers(got) == numbers(alone(prec, r, r["sweeps"], recompute_every=3))
    assert alone(prec, reqs[1], 7)["logdet"] != results[1]["logdet"]  # the recomputes show in the numbers


def test_result_after_a_step_with_a_recompute():
    """The step's recompute takes milliseconds at this size; the result read
    right after the step is the one read later, and the walker can leave."""
    require_gpu()
    r = request(21, 1024, sweeps=4, sigma=0.05)
    with pool(dsu.FP32_MIXED, recompute_every=1) as s:
        slot = add(s, r)
        s.step()
        first = s.result(slot)
        time.sleep(0.2)
        assert numbers(s.result(slot)) == numbers(first)
        s.step()
        last = s.result(slot, remove=True)
        slot = add(s, r)  # the same memory again
        s.step()
        assert numbers(s.result(slot)) == numbers(first)
    assert numbers(last) == numbers(alone(dsu.FP32_MIXED, r, 2, recompute_every=1))


def test_refused_run_counts_the_sweeps_under_way():
    """A request refused while another size is being swept: the sweep ends, is
    counted, and the walker can be read, stepped and removed."""
    require_gpu()
    long = request(31, 512, sweeps=5000, sigma=0.05)
    with pool(dsu.FP32_MIXED) as s:
        with pytest.raises(dsu.DsuError) as ex:
            s.run([long, request(32, 64, spins=3, arrival_s=0.05)])
        assert ex.value.code == dsu.EINVAL
        done = s.result(0)["sweeps_done"]
        assert 0 < done < 5000
        assert numbers(s.result(0)) == numbers(alone(dsu.FP32_MIXED, long, done))
        s.step()
        assert numbers(s.result(0, remove=True)) == numbers(alone(dsu.FP32_MIXED, long, done + 1))
        assert s.usage() == (0, 0)
