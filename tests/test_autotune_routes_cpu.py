"""The batch autotuner's candidates and the cache of the kernels before them."""
import json

import paper_1807_03249_amd.autotune as at


class _Cuda:
    @staticmethod
    def get_device_name(index):
        return "device"


class _Torch:
    cuda = _Cuda


def test_candidates_hold_the_default():
    """A plan with a grid of its own always replays its graph, so only the
    library's default (0) reaches the direct launches of small batches."""
    assert at.BATCH_BLOCKS_PER_CU[0] == 0
    assert set(at.BATCH_BLOCKS_PER_CU) >= {2, 4, 8, 16}


def test_tune_batch_tries_the_default(monkeypatch, tmp_path):
    """Every candidate reaches a plan, and winners cached for other kernels do not."""
    cache = tmp_path / "tune.json"
    key = f"|{at.batch_signature([])}"
    cache.write_text(json.dumps({f"device|choices5{key}": {
        "tune": [4, 16, 2, 2, 2], "blocks_per_cu": 8, "ms": 1.0}}))
    seen = []

    class Plan:
        def __init__(self, use_graph, tune, blocks_per_cu):
            seen.append(blocks_per_cu)

        def run(self, jobs, workspace=None):
            pass

        def close(self):
            pass

    class Torch(_Torch):
        class cuda(_Cuda):
            @staticmethod
            def synchronize():
                pass

    monkeypatch.setattr(at, "_torch", lambda: Torch)
    monkeypatch.setattr(at, "Batch", Plan)
    monkeypatch.setattr(at, "_time_events", lambda torch, fn, reps: 1.0 + len(seen))
    got = at.tune_batch([], candidates=[(4, 16, 2, 2, 1)], cache_path=str(cache), workspace=0)
    assert not got["cached"] and seen == list(at.BATCH_BLOCKS_PER_CU)
    assert got["blocks_per_cu"] == 0
