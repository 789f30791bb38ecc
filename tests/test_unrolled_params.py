"""The parameters that UnrolledADM hands to its steps, on the CPU: the step itself is
replaced by one that records its row (mu, rho, xi, alpha)."""
import pytest
import torch

from paper_1607_01650_amd import configs as C
from paper_1607_01650_amd import unrolled as U

G = C.Geometry(nx=4, ny=3, pixel_mm=1.0, n_views=2, n_bins=5, bin_mm=1.0, sod_mm=20.0, sdd_mm=40.0)


@pytest.fixture
def rows(monkeypatch):
    seen = []

    def step(f, lx, ly, g, geom, params):
        seen.append(params.detach().clone())
        return f + params.sum(), lx, ly

    monkeypatch.setattr(U, "_adm_step", step)
    return seen


def _run(model, rows):
    rows.clear()
    model(torch.zeros((1, G.n_views, G.n_bins)), use_checkpoint=False)
    return torch.stack(rows)


def test_more_steps_than_rows(rows):
    m = U.UnrolledADM(G, n_steps=3)
    m.n_steps = 5
    with pytest.raises(IndexError):
        _run(m, rows)
