"""A pause of the host while the autotuner times a candidate does not decide:
the plan that modal_init chooses by itself is kept for a batch of strings
although the host stops for 20 ms in its first timed run (100 samples take
0.03 ms on it, 0.2 ms and more on the step kernel)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_a_pause_in_one_run_does_not_decide(tmp_path, monkeypatch):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal, tune
    k = np.arange(1.0, 13.0)
    insts = [dict(kind="tension", omega=2 * np.pi * 100 * k * (1 + 0.01 * b / 600), gamma=np.full(12, 3.0),
                  x0=1e-3 / k, xm1=1e-3 / k, c=np.ones(12), lam=k ** 2, kappa=1e4) for b in range(600)]

    class Paused(modal.Sim):
        def __init__(self, *a, **kw):
            super().__init__(*a, **kw)
            self.pauses, self.runs = "waves" not in kw, 0

        def run(self, *a, **kw):
            self.runs += 1
            if self.pauses and self.runs == 2:
                time.sleep(0.02)
            return super().run(*a, **kw)

    monkeypatch.setattr(modal, "Sim", Paused)
    best = tune.autotune(insts, 44100.0, shapes=((4, 2), (8, 1)), samples=100, cache=str(tmp_path / "t.json"), split_costs=(32,))
    assert best == (0, 0, 0)
