"""The autotuner times only what changes a launch: bwd_batch, which the backward
does not read, stays at its default (no GPU: the timings are made up)."""
import itertools

import torch

from paper_2601_19489_amd import batched


class _Event:
    clock = itertools.count()

    def __init__(self, enable_timing=False):
        pass

    def record(self):
        self.at = 0

    def elapsed_time(self, other):
        return 100.0 - next(_Event.clock)   # every later candidate looks faster


class _Step:
    def run(self):
        pass

    def check_capacity(self):
        pass


def test_autotuner_does_not_search_a_knob_without_effect(monkeypatch):
    knobs = []
    monkeypatch.setattr(batched._lib, 'gs_set_tuning', lambda **k: knobs.append(k))
    monkeypatch.setattr(torch.cuda, 'Event', _Event)
    monkeypatch.setattr(torch.cuda, 'synchronize', lambda: None)
    best, table = batched.autotune(lambda tile: _Step(), bwd_batch=(32, 64, 128))
    assert [c['bwd_batch'] for c, _ in table] == [0] * len(table)
    assert best['bwd_batch'] == 0 and all(k['bwd_batch'] == 0 for k in knobs)
    # the others are searched: their last candidates win here
    assert best['fwd_batch'] == 256 and best['persist_wgs'] == 16 and best['fwd_px'] == 4
