"""The batched stages of a product at the sizes where their kernels change
shape, residue for residue equal to the CPU oracle (single ciphertexts) or to
each member computed alone (batches)."""
import numpy as np
import pytest

from paper_2305_17341_amd import inputs as I

pytestmark = pytest.mark.gpu

TINY = I.Chain("n11_stages", 11, (60,) + (40,) * 4, (60, 60))
BATCHED, LAZY, FUSED, MERGED = 1, 2, 4, 64


@pytest.mark.parametrize("chain", [TINY, I.SMALL], ids=lambda c: c.name)
@pytest.mark.parametrize("kind,n1", [("sigma", 1), ("sigma", 2), ("sigma", 16), ("tau", 1), ("tau", 8),
                                     ("transpose", 4)])
def test_giant_steps_match_oracle(oracle_mod, chain, kind, n1):
    """31, 15 and 1 giant steps of sigma, 15 and 1 of tau, 7 of the
    transposition: the steps shared out over thread groups from four on, with
    and without a step that needs no rotation"""
    from paper_2305_17341_amd import he
    n = 16
    steps = he.lintrans_rot_steps({"sigma": "Z", "tau": "T", "transpose": "G"}[kind], n, n1)
    ctx = he.chain_context(chain, seed=71)
    ctx.keygen(steps)
    o = oracle_mod.Oracle(chain.log_n, chain.q_bits, chain.p_bits, seed=71)
    o.keygen(rot_steps=steps)
    A = I.uniform_matrix(5, n)
    g = ctx.lintrans(ctx.encrypt_matrix(A, nonce=2), kind, n, n1)
    f = {"sigma": o.lt_sigma, "tau": o.lt_tau, "transpose": o.lt_transpose}[kind]
    w = f(o.encrypt(A.ravel(), nonce=2), n, n1)
    assert g.level == w.level and g.scale == w.scale
    assert np.array_equal(g.export(), w.data())


@pytest.mark.parametrize("flags", [0, LAZY | FUSED], ids=["paper", "lazy-fused"])
@pytest.mark.parametrize("chain,d,n1", [(I.SMALL, 16, 2), (I.SMALL, 16, 16), (I.MID, 32, 8)],
                         ids=["n13-n1_2", "n13-n1_16", "n14-n1_8"])
@pytest.mark.parametrize("batch", [2, 3, 5, 6, 7])
def test_batches_match_members_alone(chain, d, n1, batch, flags):
    from paper_2305_17341_amd import he
    opts = {"n1_z": n1, "n1_t": n1}
    ctx = he.chain_context(chain, seed=72)
    ctx.keygen(ctx.matmul_rot_steps(d, opts))
    a = [ctx.encrypt_matrix(I.uniform_matrix(10 + i, d), nonce=10 + i) for i in range(batch)]
    b = [ctx.encrypt_matrix(I.uniform_matrix(30 + i, d), nonce=30 + i) for i in range(batch)]
    got = ctx.matmul_batch(a, b, [d] * batch, dict(opts, flags=BATCHED | flags))
    for i in range(batch):
        alone = ctx.matmul(a[i], b[i], d, dict(opts, flags=flags))
        assert np.array_equal(got[i].export(), alone.export()), i
        err = np.max(np.abs(ctx.decrypt(got[i], d * d) - (I.uniform_matrix(10 + i, d) @ I.uniform_matrix(30 + i, d)).ravel()))
        assert err < 2.0**-15
