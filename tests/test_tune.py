"""What the autotuner times: explicit parameters of the delegate method for single
problems (a plain call runs another path), and batches that the table applies to."""
import types

import pytest

torch = pytest.importorskip("torch")
drt = pytest.importorskip("paper_2109_08219_amd")
tune = pytest.importorskip("paper_2109_08219_amd.tune")


class Keys:
    dtype, device = torch.float32, "cpu"

    def __init__(self, n):
        self.n = n

    def view(self, *_):
        return self

    def __getitem__(self, s):
        return Keys(s.stop)

    def numel(self):
        return self.n


class Event:
    def __init__(self, enable_timing):
        pass

    def record(self):
        pass

    synchronize = record

    def elapsed_time(self, other):
        return 1.0


def fake_torch():
    cuda = types.SimpleNamespace(Event=Event, synchronize=lambda: None, empty_cache=lambda: None)
    return types.SimpleNamespace(cuda=cuda, manual_seed=lambda s: None, Generator=lambda: types.SimpleNamespace(
        manual_seed=lambda s: None), randint=lambda lo, hi, size, **kw: torch.full(size, lo) if kw.get("device") == "cpu"
        else Keys(size[0]), randn=lambda n, **kw: Keys(n), empty=lambda n, **kw: Keys(n), int32=torch.int32,
        uint32=torch.uint32)


def test_single_candidates_are_explicit():
    calls = []
    fake = types.SimpleNamespace(FORM_SINGLE=0, FORM_BATCHED=1, tune_set=lambda e: None, plan=drt.plan,
                                 topk_select=lambda t, k, v, i, **kw: calls.append((t.n, k, kw)))
    tune.tune_single(fake, fake_torch(), 1, log=lambda s: None)
    assert calls and all(kw.get("mode") == 1 and kw["alpha"] >= 0 and kw["beta"] >= 1 for _, _, kw in calls)


def test_batches_are_ones_that_the_table_applies_to():
    seen = []

    class Batch:
        def __init__(self, probs):
            seen.append([(t.numel(), k) for t, k in probs])

        def run(self):
            pass

    fake = types.SimpleNamespace(FORM_SINGLE=0, FORM_BATCHED=1, tune_set=lambda e: drt.tune_set([]), Batch=Batch,
                                 batched_plan=drt.batched_plan, batched_streams=drt.batched_streams)
    saved = drt.tune_get()
    try:
        tune.tune_batched(fake, fake_torch(), 512, 1, log=lambda s: None)
    finally:
        drt.tune_set(saved)
    assert seen
    for probs in seen:
        n, k = probs[0]
        if n <= 1 << 16:
            assert not drt.batched_streams(n, k, len(probs)), (n, k, len(probs))
        else:  # split: more than a slot's share of the batch
            assert n * 512 > sum(m for m, _ in probs), (n, len(probs))
