"""Gram-Schmidt of long vectors in the Lanczos step: above 65536 elements the
partial sums of a pass are added up by a launch of their own, above 262144 a
workgroup works off several chunks of its rows; odd lengths, and more rows than
one lane group holds (16, 24 and 40 Krylov vectors)."""
import numpy as np
import pytest
import torch

from paper_1501_05504_amd import synth

pytestmark = pytest.mark.gpu

abi = pytest.importorskip("paper_1501_05504_amd.abi")

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx():
    c = abi.Context(0)
    yield c
    c.close()


def lanczos(apply, x, steps):
    """Lowest Ritz pair of `steps` plain Lanczos steps with full
    re-orthogonalisation, in torch."""
    V = [x / x.norm()]
    a, b = [], []
    for k in range(steps):
        w = apply(V[k])
        a.append(float(torch.dot(w, V[k])))
        Q = torch.stack(V)
        for _ in range(2):
            w = w - torch.mv(Q.t(), torch.mv(Q, w))
        b.append(float(w.norm()))
        V.append(w / b[-1])
    e, y = np.linalg.eigh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
    x = torch.mv(torch.stack(V[:-1]).t(), torch.tensor(y[:, 0], device=DEV))
    return e[0], x / x.norm(), e[1] - e[0]


@pytest.mark.parametrize("ml, d, mr", [(128, 4, 128), (129, 4, 129), (129, 1, 511), (256, 4, 256), (257, 4, 257), (257, 1, 1021),
                                       (420, 2, 700)])
@pytest.mark.parametrize("steps", [16, 24, 40])
def test_lanczos_of_long_vectors(ctx, ml, d, mr, steps):
    """The Ritz value and vector after one run of `steps` products equal those of
    a plain Lanczos run.  Rounding perturbs the tridiagonal matrix by some 1e-14 of
    its norm: the value agrees to 1e-12 of that, the vector to 1e-12 of the norm
    over the gap to the next Ritz value."""
    gen = torch.Generator(device=DEV).manual_seed(ml + mr)
    rnd = lambda *s: torch.randn(*s, generator=gen, dtype=torch.float64, device=DEV)
    w = 3
    sym = lambda x: ((x + x.transpose(0, 2)) / 2).contiguous()
    L, R, W = sym(rnd(ml, w, ml)), sym(rnd(mr, w, mr)), rnd(w, w, d, d)
    W = ((W + W.transpose(2, 3)) / 2).contiguous()
    x = rnd(ml, d, mr)

    def apply(v):
        T = torch.matmul(L.reshape(ml * w, ml), v.reshape(ml, d * mr)).reshape(ml, w, d, mr)
        T = torch.tensordot(T, W, dims=([1, 2], [0, 3])).permute(0, 3, 2, 1).reshape(ml * d, w * mr).contiguous()
        return torch.matmul(T, R.reshape(mr, w * mr).t().contiguous()).reshape(-1)
    ref, vec, gap = lanczos(apply, x.reshape(-1).clone(), steps)
    th, nmv, _ = ctx.lanczos(L, W, R, x, tol=1e-30, kmax=steps, max_matvecs=steps)
    x = x.reshape(-1)
    assert nmv == steps and abs(float(x.norm()) - 1) < 1e-13
    assert abs(th - ref) <= 1e-12 * abs(ref)
    x = x * torch.sign(torch.dot(x, vec))
    assert float((x - vec).norm()) <= 1e-12 * abs(ref) / gap


def test_long_vectors_in_the_captured_step(ctx):
    """The step of the block sweeps that reads its index on the device (captured
    once, replayed): a Heisenberg chain of 20 sites with one trivial sector has
    vectors of up to 512 x 2 x 600 elements.  Its energy is not above that of Sz
    sectors with 96 states (vectors below 65536) but for the solver's tolerance,
    and not below it by more than their truncation, some 1e-8, can cost."""
    l = 20
    mpo = abi.heisenberg_mpo(l)
    none = np.zeros_like(np.array(abi.SPIN_HALF_CHARGES))

    def run(phys, chan, m, sweeps):
        tensors, secs = synth.random_symmetric_mps(l, phys, [0], m, seed=5)
        st = abi.State(mpo, tensors, m, device=DEV)
        sym = abi.Symmetry(phys, abi.mpo_bond_charges(mpo, chan), secs)
        params = abi.sweep_params(alpha=1e-3, e_before=ctx.prepare_blocks(st, sym))
        for _ in range(sweeps):
            _, stats, _ = ctx.sweep_blocks(st, sym, params, use_graph=True)
        return stats.energy
    chan = abi.mpo_spin_charges(1)
    ref = run(np.array(abi.SPIN_HALF_CHARGES), chan, 96, 8)
    e = run(none, np.zeros_like(chan), 600, 4)
    assert ref - 1e-6 < e < ref + 1e-10
