"""Terms of Eq. tx2 that the amplitude-dependent blocks carry, checked on random tensors with the
symmetries that make it exact (one k point; the k-blocked sums are the same sums split by momentum)."""
import numpy as np
import pytest


def _c(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _pab(z):
    return z - z.transpose(0, 1, 3, 2)


def _pij(z):
    return z - z.transpose(1, 0, 2, 3)


@pytest.mark.parametrize("o,v,seed", [(1, 2, 1), (3, 4, 2), (4, 3, 3)])
def test_one_body_terms_of_x2(o, v, seed):
    """P(ij)P(ab) [1/2 x_ijae F_be - 1/2 x_imab F_mj] = P(ij)P(ab) of the ring product with the off-diagonal
    elements + (F_aa + F_bb - F_ii - F_jj) x_ijab; transposed with the same diagonal."""
    rng = np.random.default_rng(seed)
    x = _pij(_pab(_c(rng, o, o, v, v)))
    fbe, fmj = _c(rng, v, v), _c(rng, o, o)
    old = _pij(_pab(0.5 * np.einsum('ijae,be->ijab', x, fbe) - 0.5 * np.einsum('imab,mj->ijab', x, fmj)))
    db, dj = np.diag(fbe), np.diag(fmj)
    w = (0.5 * np.einsum('mj,be->mebj', np.eye(o), fbe - np.diag(db))
         - 0.5 * np.einsum('be,mj->mebj', np.eye(v), fmj - np.diag(dj)))
    d = db[:, None] + db[None, :] - dj[:, None, None, None] - dj[None, :, None, None]
    new = _pij(_pab(np.einsum('imae,mebj->ijab', x, w))) + d * x
    # sums of at most 4 (o + v) + 4 products of numbers below 10, in double
    assert np.abs(old - new).max() < 1e-12 * max(1.0, np.abs(old).max())
    # the quarter that joins Z before P(ij)P(ab)
    assert np.abs(_pij(_pab(0.25 * d * x)) - d * x).max() < 1e-12 * max(1.0, np.abs(d * x).max())


@pytest.mark.parametrize("o,v,seed", [(2, 2, 4), (3, 4, 5), (4, 3, 6)])
def test_x1_terms_in_one_block(o, v, seed):
    """Under P(ij)P(ab): - (U_ianf x_jf) t_nb = x_ie (U_jane t_nb);
    (x_je g_mnie - x_ie g_mnje) tau_mnab / 8 = - x_ie (g_mnje tau_mnab) / 4; - G_ijbm x_ma = G_ijan x_nb."""
    rng = np.random.default_rng(seed)
    x1, t1 = _c(rng, o, v), _c(rng, o, v)
    u = _c(rng, o, v, o, v)
    g = _c(rng, o, o, o, v)
    g = g - g.transpose(1, 0, 2, 3)
    tau = _pij(_pab(_c(rng, o, o, v, v)))
    gg = _c(rng, o, o, v, o)
    vx = np.einsum('je,mnie->ijmn', x1, g) - np.einsum('ie,mnje->ijmn', x1, g)
    pairs = [
        (-np.einsum('ianf,jf,nb->ijab', u, x1, t1), np.einsum('ie,jane,nb->ijab', x1, u, t1)),
        (np.einsum('ijmn,mnab->ijab', vx, tau) / 8, -np.einsum('ie,mnje,mnab->ijab', x1, g, tau) / 4),
        (-np.einsum('ijbm,ma->ijab', gg, x1), np.einsum('ijan,nb->ijab', gg, x1)),
    ]
    for old, new in pairs:
        a, b = _pij(_pab(old)), _pij(_pab(new))
        assert np.abs(a - b).max() < 1e-12 * max(1.0, np.abs(a).max())
