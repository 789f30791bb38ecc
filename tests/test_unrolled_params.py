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


def _doubled(self, k):
    mu, rho, xi, alpha = (torch.exp(t[k]).float() for t in (self.log_mu, self.log_rho, self.log_xi, self.log_alpha))
    return 2 * mu, rho, xi, (k + 1) * alpha


@pytest.mark.parametrize("where", ["instance", "other instance's", "class", "subclass"])
def test_params_of_replaced(rows, monkeypatch, where):
    m = U.UnrolledADM(G, n_steps=3, mu=0.5, alphas=[1e-4, 2e-4, 3e-4])
    plain = _run(m, rows)
    want = plain * torch.tensor([[2.0, 1.0, 1.0, k + 1.0] for k in range(3)])
    if where == "instance":
        m.params_of = lambda k: _doubled(m, k)
    elif where == "other instance's":
        other = U.UnrolledADM(G, n_steps=3, mu=1.0, alphas=[1e-4, 4e-4, 9e-4])
        m.params_of = other.params_of
    elif where == "class":
        monkeypatch.setattr(U.UnrolledADM, "params_of", _doubled)
    else:
        sub = type("Sub", (U.UnrolledADM,), {"params_of": _doubled})
        m = sub(G, n_steps=3, mu=0.5, alphas=[1e-4, 2e-4, 3e-4])
    torch.testing.assert_close(_run(m, rows), want, rtol=1e-6, atol=0)


# Parameter tables that params_of takes, though they are not four float64 vectors of one length.
@pytest.mark.parametrize("change", ["longer alphas", "float32", "list", "column", "gone"])
def test_tables_of_other_forms(rows, change):
    m = U.UnrolledADM(G, n_steps=3, mu=0.5, alphas=[1e-4, 2e-4, 3e-4, 4e-4, 5e-4][:5 if change == "longer alphas" else 3])
    if change == "float32":  # each table keeps its own precision
        m.log_rho = torch.nn.Parameter(m.log_rho.detach().float())
    elif change == "list":
        mu = m.log_mu.detach()
        del m.log_mu
        m.log_mu = torch.nn.ParameterList([torch.nn.Parameter(v.clone()) for v in mu])
    elif change == "column":
        m.log_xi = torch.nn.Parameter(m.log_xi.detach()[:, None][:, 0])
    elif change == "gone":
        rho, m.params_of = m.log_rho.detach(), None
        del m.log_rho
        m.params_of = lambda k: (torch.exp(m.log_mu[k]).float(), torch.exp(rho[k]).float(),
                                 torch.exp(m.log_xi[k]).float(), torch.exp(m.log_alpha[k]).float())
    assert torch.equal(_run(m, rows), torch.stack([torch.stack(m.params_of(k)) for k in range(3)]))
