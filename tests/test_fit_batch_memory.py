"""Strike projections of many plates at once: the memory they take does not
grow with their number, and the values are those of each plate alone."""
import tracemalloc

import numpy as np


def test_many_plates_with_a_wide_strike():
    from paper_2505_05940_amd import fit
    setup = fit.PlateSetup(n_t=12, n_in=12, strike=(0.5, 0.5, 1e-3, 0.5))  # the whole grid
    a = np.random.default_rng(1).uniform(0.4, 1.4, 700)
    fit.excitations(setup, a[:2])
    tracemalloc.start()
    x0, c = fit.excitations(setup, a)
    peak = tracemalloc.get_traced_memory()[1]
    tracemalloc.stop()
    assert x0.shape == c.shape == (700, 12)
    assert peak < 300e6, peak  # 700 boxes of 30000 points and their temporaries: 700 MB and more
    for b in (0, 1, 82, 83, 84, 699):
        one = fit._excitation(setup, a[b])
        for got, ref in zip((x0[b], c[b]), one):
            assert np.allclose(got, ref, rtol=1e-12, atol=1e-13 * np.abs(ref).max())
