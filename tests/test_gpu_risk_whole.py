"""hilore_unit_exposure_risk on units of one row chunk (at most 2048 rows), which one
launch finishes, against the two-launch form of the same rows.

A row of zeros appended outside the mask makes a second chunk whose sums are all
zero, so the folded results must equal the single launch's bit for bit.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def score(hl, coeff, mask, rows, units, noalloc=False):
    o = torch.full((3, len(units)), float("nan"), device="cuda")
    call = hl.hilore_unit_exposure_risk_noalloc if noalloc else hl.hilore_unit_exposure_risk
    call(coeff, mask, rows, units, 1e-8, 1e-8, o[0], o[1], o[2])
    return o


@pytest.mark.parametrize("n_units", [1, 96, 97, 130])
@pytest.mark.parametrize("masked", [0, 0.3, 1], ids=["all", "some", "none"])
def test_one_chunk_matches_two(hl, n_units, masked):
    rows, longer = 2048, 2049
    g = torch.Generator(device="cuda").manual_seed(n_units)
    ss = torch.zeros(2, n_units, 2052, device="cuda")
    ss[0, :, :rows] = 100.0 * torch.rand((n_units, rows), generator=g, device="cuda")
    ss[1, :, :rows] = 1e-2 * torch.rand((n_units, rows), generator=g, device="cuda")
    coeff = torch.zeros(2052, device="cuda")
    coeff[:rows] = 1e-4 * torch.randn(rows, generator=g, device="cuda")
    mask = torch.zeros(2064, dtype=torch.uint8, device="cuda")
    mask[:rows] = (torch.rand(rows, generator=g, device="cuda") >= masked).to(torch.uint8)
    cols = [128 * (1 + u % 7) for u in range(n_units)]

    def units(r):
        return [hl.unit_desc(row_ss_x=ss[0, u, :r], row_ss_err=ss[1, u, :r], rows=r, cols=cols[u],
                             ld=cols[u]) for u in range(n_units)]

    one = score(hl, coeff[:rows], mask[:rows], rows, units(rows))
    two = score(hl, coeff[:longer], mask[:longer], longer, units(longer))
    assert torch.equal(one, two) and bool(torch.isfinite(one).all())
    assert torch.equal(one, score(hl, coeff[:rows], mask[:rows], rows, units(rows), noalloc=True))
