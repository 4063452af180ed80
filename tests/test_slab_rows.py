"""The planner's smallest slab: instances below 4 MB are cut into slabs of at
least four in-plane rows (or 128 KB of rows), whatever the number of
workgroups, and are whole where that leaves nothing to cut.  Counted from the
rule itself: row bytes 4 n_t (n_t rounded up to 4) + 4096."""
import numpy as np
import pytest


def inst(n_t, n_in):
    H = np.zeros((n_in, n_t, n_t), np.float32)
    return dict(kind="vk", omega=np.linspace(100, 5000, n_t), gamma=np.ones(n_t), x0=np.zeros(n_t),
                xm1=np.zeros(n_t), c=np.ones(n_t), Ht=H)


@pytest.mark.parametrize("n_t,n_in,units", [
    (64, 64, 16),    # 64 rows in fours
    (50, 50, 13),    # 50 rows: 12.5
    (72, 66, 17),
    (120, 60, 20),   # 61.7 KB a row: three rows to 128 KB
    (200, 20, 20),   # 164 KB a row: single rows
    (160, 5, 3),     # 106 KB a row, two rows, five of them
    (40, 40, 1),     # below the bound on cut instances
    (100, 100, 100),  # 4.4 MB: above the rule
])
def test_lone_plates_are_not_cut_finer(n_t, n_in, units):
    from paper_2505_05940_amd import modal
    assert modal.plan([inst(n_t, n_in)], 256)["units"] == units


@pytest.mark.parametrize("n", [50, 64, 80])
def test_few_plates_share_the_rule(n):
    from paper_2505_05940_amd import modal
    assert modal.plan([inst(n, n)] * 3, 768)["units"] <= 3 * -(-n // 4)
