"""The batched host side of a plate fit (instances and chain rule of all plates
at once) against the one-plate functions, which the oracle pins."""
import numpy as np
import pytest


@pytest.mark.parametrize("n,grid,strike", [(1, (200, 150), (0.37, 0.61, 1e-3, 0.1)), (24, (96, 72), (0.37, 0.61, 1e-3, 0.1)),
                                           (60, (64, 64), (0.02, 0.97, 2e-3, 0.3)), (9, (8, 5), (0.5, 0.5, 1e-3, 0.05))])
def test_batch_matches_single_plates(n, grid, strike):
    from paper_2505_05940_amd import fit
    setup = fit.PlateSetup(n_t=n, n_in=n + 1, proj_grid=grid, strike=strike)
    rng = np.random.default_rng(n)
    B = 7
    th = np.stack([rng.uniform(3, 9, B), rng.uniform(1, 4, B), rng.uniform(0.31, 1.5, B), rng.uniform(0.5, 2, B),
                   rng.uniform(1e-4, 1e-3, B)], 1)
    insts, lam, omega = fit.plate_instances_shared(setup, th)
    g = {k: [rng.normal(size=n) for _ in range(B)] for k in ("omega", "gamma", "c", "x0", "xm1")}
    g["row"] = [rng.normal(size=n + 1) for _ in range(B)]
    g["scale"], g["theta"] = rng.normal(size=B), np.zeros(B)
    got = fit.chain_rules(setup, th, lam, omega, g)
    for b in range(B):
        one = fit.plate_instance_shared(setup, th[b])
        for k in ("omega", "gamma", "lam", "x0", "xm1", "c", "h_row_scale", "zeta2"):
            assert np.allclose(insts[b][k], one[k], rtol=1e-12, atol=1e-13 * np.abs(one[k]).max()), k
        assert insts[b]["Ht"] is one["Ht"] and np.array_equal(insts[b]["mode_class"], one["mode_class"])
        ref = fit.chain_rule(setup, th[b], one, {k: v[b] for k, v in g.items()})
        # the strike's aspect derivative is a difference over 2e-6 of values
        # equal to a few 1e-16: 1e-9 of its own scale
        assert np.allclose(got[b], ref, rtol=1e-9, atol=1e-9 * np.abs(ref).max())
