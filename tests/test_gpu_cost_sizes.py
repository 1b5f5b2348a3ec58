"""The unravelling cost's exponential and its Frechet derivative at their edges: part-filled
groups of states, zero and tiny generators (no squaring), large ones (many squarings).
Tolerances: a squaring doubles the relative error, 2^s is about 4 ||H||_1 and ||H||_1 a few times
the parameters' scale, so the bounds of test_gpu_cost.py grow with 1 + scale."""
import numpy as np
import pytest

from oracle import cost as CO
from paper_2508_05745_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,scale", [(1, 0.0), (15, 1e-7), (16, 1.0), (17, 6.0), (33, 40.0)])
@pytest.mark.parametrize("kind", [0, 1])
def test_cost_generator_sizes(batch, scale, kind):
    import torch

    from paper_2508_05745_amd import mpsb as M
    th = I.random_two_site_states(batch, 3, 5, seed=4100, dtype=np.complex128)
    rng = np.random.default_rng(4101)
    params = scale * rng.standard_normal((batch, 16))
    uref = np.stack([I.haar_unitary(rng, 4) for _ in range(batch)])
    k = I.random_channel(4, 4102)
    pp, uu = torch.as_tensor(params).cuda(), torch.as_tensor(uref).cuda()
    f, rho, k4 = M.unravel_cost(torch.as_tensor(th).cuda(), k, pp, uu, kind)
    g = M.unravel_cost_grad(rho, k4, pp, uu, kind, None).cpu().numpy()
    for b in range(batch):
        r = CO.rho_from_theta(th[b])
        f_ref, g_ref = CO.grad_torch(r / np.trace(r).real, k, params[b], uref[b], kind)
        assert abs(f[b].item() - f_ref) < 1e-12 * (1 + scale)
        assert np.linalg.norm(g[b] - g_ref) <= 1e-10 * (1 + scale) * max(1.0, np.linalg.norm(g_ref))


@pytest.mark.parametrize("kind", [0, 1])
def test_cost_generator_norm_at_a_power_of_two(kind):
    """Generators of column norm 1 whose four terms sum to 1 or to 1 + 2^-52 by the order of the
    addition: the number of squarings jumps there, and every lane of a state must take the same."""
    import torch

    from paper_2508_05745_amd import mpsb as M
    # columns 0 .. 3 of H take (d, o, 0, z) from the diagonal entry and two real couplings
    params = np.zeros((24, 16))
    for b in range(24):
        d, o, z = [(0.2, 7 * 0.1, 0.1), (0.1, 0.2, 7 * 0.1), (7 * 0.1, 0.1, 0.2)][b % 3]
        col, scale = (b // 3) % 4, [1.0, 4.0][b // 12]
        rows = [x for x in range(4) if x != col]
        pair = {(0, 1): 4, (0, 2): 5, (0, 3): 6, (1, 2): 7, (1, 3): 8, (2, 3): 9}
        params[b, col] = scale * d
        params[b, pair[tuple(sorted((col, rows[0])))]] = scale * o
        params[b, pair[tuple(sorted((col, rows[2])))]] = scale * z
    th = I.random_two_site_states(24, 3, 5, seed=4110, dtype=np.complex128)
    rng = np.random.default_rng(4111)
    uref = np.stack([I.haar_unitary(rng, 4) for _ in range(24)])
    k = I.random_channel(4, 4112)
    pp, uu = torch.as_tensor(params).cuda(), torch.as_tensor(uref).cuda()
    f, rho, k4 = M.unravel_cost(torch.as_tensor(th).cuda(), k, pp, uu, kind)
    g = M.unravel_cost_grad(rho, k4, pp, uu, kind, None).cpu().numpy()
    for b in range(24):
        r = CO.rho_from_theta(th[b])
        f_ref, g_ref = CO.grad_torch(r / np.trace(r).real, k, params[b], uref[b], kind)
        assert abs(f[b].item() - f_ref) < 1e-12 * (1 + np.abs(params[b]).max()), b
        assert np.linalg.norm(g[b] - g_ref) <= 1e-10 * (1 + np.abs(params[b]).max()) * max(1.0, np.linalg.norm(g_ref)), b
