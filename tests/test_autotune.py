"""What the autotuner times, on the host: the library's own choice is among the
candidates, so that a tuned call is not slower than one that names nothing."""

import pytest
import torch

from paper_2606_00444_amd import api, autotune


class _Bvh:
    n = 500


@pytest.fixture
def timed(monkeypatch):
    """Calls of the query functions instead of launches; their times by `cost`."""
    calls = []
    monkeypatch.setattr(autotune, "_key", lambda *a, **k: "key")
    monkeypatch.setattr(api, "closest_point_query", lambda *a, **kw: calls.append(kw))
    monkeypatch.setattr(api, "nearest_point_query", lambda *a, **kw: calls.append(kw))
    return calls


def _own_choice(kw):
    """Whether these arguments leave the traversal to the library: what rules out its scan
    and its order is a kernel, batch, work counter, wave count or order asked for."""
    return (kw.get("kernel") in (None, "auto") and not any(kw.get(k) for k in ("batch", "dynamic", "waves"))
            and kw.get("order") is None and kw.get("counters") is None)


@pytest.mark.parametrize("tune", [autotune.tune_closest, autotune.tune_nearest])
@pytest.mark.parametrize("order", [None, torch.arange(4, dtype=torch.int32)])
def test_the_default_call_is_timed_and_can_win(tune, order, timed, monkeypatch):
    def cost(run, reps):
        run()
        return 1.0 if _own_choice(timed[-1]) else 2.0
    monkeypatch.setattr(autotune, "_graph_time", cost)
    res = tune(_Bvh(), None, torch.zeros(3, 4), order=order, use_cache=False)
    assert sum(_own_choice(kw) for kw in timed) >= 1
    assert res["ms"] == 1.0 and res["order"] == "given"
    assert _own_choice(autotune.options(res, order))


def test_a_named_traversal_that_wins_is_returned(timed, monkeypatch):
    def cost(run, reps):
        run()
        return 1.0 if timed[-1]["kernel"] == "batch" and timed[-1]["batch"] == 8 and timed[-1]["dynamic"] else 2.0
    monkeypatch.setattr(autotune, "_graph_time", cost)
    res = autotune.tune_closest(_Bvh(), None, torch.zeros(3, 4), use_cache=False)
    assert autotune.options(res) == {"kernel": "batch", "batch": 8, "seed": True, "dynamic": True}


@pytest.mark.parametrize("own,kept", [(1.02, True), (1.05, False)])
def test_the_default_call_is_kept_unless_clearly_slower(own, kept, timed, monkeypatch):
    """Tuned on cold queries, a choice is used with hints too: a named batch that wins by less
    than two runs differ would fix what the default follows."""
    def cost(run, reps):
        run()
        kw = timed[-1]
        return own if _own_choice(kw) else 1.0 if kw["kernel"] == "batch" and kw["batch"] == 8 and not kw["dynamic"] else 2.0
    monkeypatch.setattr(autotune, "_graph_time", cost)
    res = autotune.tune_closest(_Bvh(), None, torch.zeros(3, 4), use_cache=False)
    assert res["auto"] is kept and res["ms"] == (own if kept else 1.0)


def test_choices_of_earlier_candidates_are_not_reused(tmp_path, monkeypatch):
    """A stored choice is found by a key that names the candidates' format."""
    class Props:
        name = gcnArchName = "gfx950"
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: Props)
    key = autotune._key("closest", _Bvh(), torch.zeros(3, 4), False)
    assert key.startswith(autotune.FORMAT + "|") and key != "gfx950|closest|n=500|q=4|ordered=0"


def test_the_untuned_plan_is_timed_and_can_win(monkeypatch):
    """tune_batch times the plan as BatchPlan configures it by default, whatever the scenes'
    picks, and applies it if it is the fastest."""
    class Plan:
        plan = torch.zeros(1)
        scenes = [{"frames": torch.zeros(1, 3, 9), "faces": torch.zeros(3, n, dtype=torch.int32),
                   "gface": torch.zeros(5), "queries": torch.zeros(3, 40)} for n in (7, 8)]
        tried = []

        def configure(self, *, batch=0, seed=True, gauss_tile=2048, query_tile=256, per_scene=None):
            own = [(p.get("batch") or batch, seed if p.get("seed") is None else p["seed"])
                   for p in per_scene or [{}] * len(self.scenes)]
            self.now = (gauss_tile, query_tile, own)

        def run(self):
            self.tried.append(self.now)

    class Props:
        name = gcnArchName = "gfx950"

    untuned = (2048, 256, [(0, True), (0, True)])
    plan = Plan()

    def cost(run, reps):
        run()
        return 1.0 if plan.now == untuned else 2.0
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: Props)
    monkeypatch.setattr(api, "lbvh_build", lambda v, f: None)
    monkeypatch.setattr(autotune, "tune_closest", lambda *a, **kw: {"batch": 4, "seed": False})
    monkeypatch.setattr(autotune, "_graph_time", cost)
    res = autotune.tune_batch(plan, use_cache=False)
    assert untuned in plan.tried and (2048, 256, [(4, False), (4, False)]) in plan.tried
    assert plan.now == untuned and res["ms"] == 1.0
