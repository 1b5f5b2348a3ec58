"""unravel_opt at the sizes where its kernel can go wrong: the edges of a wave, one to four Kraus
operators, operators too weak for squares of their overlaps, basis states.  As in
test_gpu_unravel.py the optimum is checked through what is unique, with the same tolerances."""
import numpy as np
import pytest

from oracle import unravel as OU
from paper_2508_05745_amd import inputs as I

pytestmark = pytest.mark.gpu


def _channel(name):
    if name.startswith("random"):
        return I.random_channel(int(name[-1]), 6100 + int(name[-1]))
    return I.amplitude_damping(float(name.split("_")[1]))


@pytest.mark.parametrize("name,items", [("random_r1", 1), ("random_r2", 63), ("random_r3", 64), ("random_r4", 65),
                                        ("ad_1e-14", 65), ("ad_1e-280", 64)])
def test_unravel_opt_sizes(name, items):
    from paper_2508_05745_amd import mpsb as M
    k = _channel(name)
    rho = np.stack([I.random_density_matrices(1, 1300 + t, rank=1 if t % 5 == 0 else 2)[0] for t in range(items)])
    if items > 2:
        rho[1], rho[2] = np.diag([1.0, 0.0]), np.eye(2) / 2
    U, p, eof = (x.cpu().numpy() for x in M.unravel_opt(rho, k))
    for b in range(items):
        ref = OU.optimal_mixing(rho[b], k)
        assert abs(eof[b] - ref["eof"]) < 1e-12, (b, eof[b], ref["eof"])
        kp = np.einsum("ji,iab->jab", U[b], k)
        assert np.abs(sum(x.conj().T @ x for x in kp) - np.eye(2)).max() < 1e-12
        pj, eav = OU.average_entanglement(rho[b], kp)
        assert abs(eav - ref["eof"]) < 1e-11, (b, eav, ref["eof"])
        assert np.abs(pj - p[b]).max() < 1e-13
        assert abs(p[b].sum() - 1) < 1e-13


@pytest.mark.parametrize("r,seed", [(3, 5003), (3, 7003), (4, 6104), (4, 7004)])
def test_event_mixings_of_product_states(r, seed):
    """Basis states make Kraus columns parallel, and the rotations shrink their remainder until its
    square underflows: the recorded mixings of gate and idle events must stay isometries (1e-12,
    as above), or the branch weights no longer sum to one.  Layer 0 acts on |0...0> by identities,
    the others on product states."""
    import torch

    from paper_2508_05745_amd import mpsb as M
    n, depth, n_traj = 5, 3, 64
    c = I.brickwork(n, depth, seed + 1, I.random_channel(r, seed), idle_noise=True)
    rng = np.random.default_rng(seed + 2)
    for l in range(depth):
        for i in range(len(c.pairs(l))):
            c.gates[l, i] = np.eye(4) if l == 0 else np.kron(I.haar_unitary(rng, 2), I.haar_unitary(rng, 2))
    b = M.Batch(n_traj, n, 4, M.FP64, 31)
    b.set_circuit(c, M.OPTIMAL)
    w = torch.zeros((n_traj, n, 4, 4), dtype=torch.complex128, device="cuda")
    for l in range(depth):
        b.apply_layer(l, w_record=w)
        u = w.cpu().numpy()[..., :r]
        err = np.abs(np.einsum("tqji,tqjk->tqik", u.conj(), u) - np.eye(r)).max(axis=(2, 3))
        assert err.max() < 1e-12, (l, np.unravel_index(err.argmax(), err.shape), err.max())
    b.sync()
    b.close()
