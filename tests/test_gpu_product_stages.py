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


@pytest.mark.parametrize("flags", [0, LAZY, LAZY | FUSED], ids=["paper", "lazy", "lazy-fused"])
@pytest.mark.parametrize("chain,n1", [(TINY, 2), (TINY, 16), (I.SMALL, 1), (I.SMALL, 4)],
                         ids=["n11-n1_2", "n11-n1_16", "n13-n1_1", "n13-n1_4"])
def test_shift_blocks_match_oracle(oracle_mod, chain, n1, flags):
    """16, 8, 4 and 1 shift blocks: bases stacked in groups of eight, all
    shifts of a group through one key inner product launch and ModDown; with
    the ring sizes whose conversions are not fused"""
    from paper_2305_17341_amd import he
    n = 16
    opts = {"n1_z": n1, "n1_t": n1}
    ctx = he.chain_context(chain, seed=73)
    steps = ctx.matmul_rot_steps(n, opts)
    ctx.keygen(steps)
    o = oracle_mod.Oracle(chain.log_n, chain.q_bits, chain.p_bits, seed=73)
    o.keygen(rot_steps=steps)
    A, B = I.uniform_matrix(1, n), I.uniform_matrix(2, n)
    g = ctx.matmul(ctx.encrypt_matrix(A, nonce=1), ctx.encrypt_matrix(B, nonce=2), n, dict(opts, flags=flags))
    w = o.matmul(o.encrypt(A.ravel(), nonce=1), o.encrypt(B.ravel(), nonce=2), n, n1, n1, lazy=bool(flags & LAZY),
                 fused_rescale=bool(flags & FUSED))
    assert g.level == w.level and g.scale == w.scale
    assert np.array_equal(g.export(), w.data())


@pytest.mark.parametrize("chain", [I.SMALL, I.MID, I.SERVE15, I.LARGE], ids=lambda c: c.name)
@pytest.mark.parametrize("inverse", [False, True], ids=["forward", "inverse"])
def test_transforms_of_few_and_many_limbs(oracle_mod, chain, inverse):
    """few limbs take four values per thread, more than 1024 tiles of 4096
    words sixteen: the same residues, the oracle's on a limb of each modulus
    size (residues 0, 1 and q - 1 among the values)"""
    from paper_2305_17341_amd import he
    ctx = he.chain_context(chain, seed=74)
    N, nm = ctx.N, len(ctx.moduli)
    many = 1024 * 4096 // N + 3
    g = np.random.default_rng(9)
    mods = [k % nm for k in range(many)]
    x = np.stack([g.integers(0, ctx.moduli[m], size=N, dtype=np.uint64) for m in mods])
    x[:, 0], x[:, 1], x[:, N - 1] = 0, 1, [ctx.moduli[m] - 1 for m in mods]
    got = ctx.ntt_limbs(x, mods, inverse)
    for k0 in range(0, many, 60):
        few = ctx.ntt_limbs(x[k0:k0 + 60], mods[k0:k0 + 60], inverse)
        assert np.array_equal(few, got[k0:k0 + 60])
    o = oracle_mod.Oracle(chain.log_n, chain.q_bits, chain.p_bits, seed=74)
    for k in (0, 1, nm - 1):
        assert np.array_equal((o.intt if inverse else o.ntt)(mods[k], x[k]), got[k])


@pytest.mark.parametrize("log_n", [10, 11, 13, 16])
def test_embedding_passes_match_oracle(oracle_mod, log_n):
    """the encoder's two FFT passes from one to seven stages in the second,
    messages of one slot to all of them; decryption returns the message"""
    from paper_2305_17341_amd import he
    ch = I.Chain("emb", log_n, (60, 40), (60,))
    ctx = he.chain_context(ch, seed=75)
    ctx.keygen([])
    o = oracle_mod.Oracle(log_n, ch.q_bits, ch.p_bits, seed=75)
    for n in (1, 2, 64, ctx.slots):
        z = np.random.default_rng(n).uniform(-1, 1, n)
        assert np.array_equal(ctx.encode(z, 2.0**40), o.encode(z, 2.0**40))
        got = ctx.decrypt(ctx.encrypt(z, nonce=n))
        assert np.max(np.abs(got - np.resize(z, ctx.slots))) < 2.0**-15


def test_plaintexts_encoded_together():
    """some nine thousand messages encoded in batches (the diagonals of three
    permutations at twelve levels): every transform returns the permuted matrix"""
    from paper_2305_17341_amd import he
    n = 128
    ch = I.Chain("emb16", 16, (60,) + (40,) * 12, (60,))
    ctx = he.chain_context(ch, seed=76)
    steps = set()
    for kind in "ZTG":
        steps |= set(he.lintrans_rot_steps(kind, n, 16))
    ctx.keygen(sorted(steps))
    A = I.uniform_matrix(8, n)
    i, j = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    want = {"sigma": A[i, (i + j) % n], "tau": A[(i + j) % n, j], "transpose": A.T}
    x = ctx.encrypt_matrix(A, nonce=3)
    for level in range(1, 13):
        at = ctx.drop(x, level)
        for kind, w in want.items():
            got = ctx.decrypt(ctx.lintrans(at, kind, n, 16), n * n)
            assert np.max(np.abs(got - w.ravel())) < 2.0**-15, (kind, level)


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("level,v_level", [(4, 4), (3, 4), (2, 2)])
def test_power_blocks_together_match_oracle(oracle_mod, axis, level, v_level):
    """three by three blocks alike (one batch a stage), the vector's level
    above the blocks', and too low for a batch along one of the axes"""
    from oracle import power as P
    from paper_2305_17341_amd import he
    n, k, ch = 4, 3, TINY
    ctx = he.chain_context(ch, seed=77)
    ctx.keygen(he.power_rot_steps(n))
    o = oracle_mod.Oracle(ch.log_n, ch.q_bits, ch.p_bits, seed=77)
    o.keygen(rot_steps=he.power_rot_steps(n))
    X = I.uniform_matrix(3, n * k)
    cov = X @ X.T / (n * k)
    blocks = [cov[r * n:(r + 1) * n, c * n:(c + 1) * n] for r in range(k) for c in range(k)]
    reps = P.replicate(I.rng(4).uniform(-0.3, 0.3, n * k), k, n, axis)
    gC = [ctx.encrypt_matrix(b, level, nonce=100 + i) for i, b in enumerate(blocks)]
    oC = [P.Box(o.encrypt(b.ravel(), level, nonce=100 + i)) for i, b in enumerate(blocks)]
    gV = [ctx.encrypt_matrix(b, v_level, nonce=200 + i) for i, b in enumerate(reps)]
    oV = [P.Box(o.encrypt(b.ravel(), v_level, nonce=200 + i)) for i, b in enumerate(reps)]
    ref, hp = he.Refresher(ctx, 1 << 40), P.HePower(o, n, nonce0=1 << 40)
    gV, g_axis = ctx.power_step(gC, k, n, gV, axis, 1, 2.0, False, ref)
    oV, o_axis = hp.step(oC, k, oV, axis, 1, 2.0, False)
    assert g_axis == o_axis and ref.count == hp.refreshes
    for i in range(k):
        assert gV[i].level == oV[i].ct.level and gV[i].scale == oV[i].ct.scale
        assert np.array_equal(gV[i].export(), oV[i].ct.data()), i


@pytest.mark.parametrize("bits", [(60, 46, 41, 40, 33), (45, 45, 45, 45, 45), (60, 40, 32, 38, 46)], ids=str)
def test_key_words_of_all_sizes_match_oracle(oracle_mod, bits):
    """switching keys over moduli of 32 to 46 bits (packed in a byte or two
    above 32) and 60: a rotation, a product, hoisted rotations and a transform"""
    from paper_2305_17341_amd import he
    n, ch = 16, I.Chain("keys", 12, bits, (60, 46))
    steps = sorted(set(he.lintrans_rot_steps("Z", n, 4)) | {1, 3, -5})
    ctx = he.Context(ch.log_n, ch.q_bits, ch.p_bits, 30.0, seed=78)
    ctx.keygen(steps)
    o = oracle_mod.Oracle(ch.log_n, ch.q_bits, ch.p_bits, log2_scale=30.0, seed=78)
    o.keygen(rot_steps=steps)
    A = I.uniform_matrix(6, n)
    x, y = ctx.encrypt_matrix(A, nonce=1), o.encrypt(A.ravel(), nonce=1)
    assert np.array_equal(ctx.rotate(x, 3).export(), o.rotate(y, 3).data())
    assert np.array_equal(ctx.mult(x, x).export(), o.mult(y, y).data())
    many = ctx.rotate_many([x, x], [1, 3, -5])
    for r, s in enumerate([1, 3, -5]):
        for member in many:
            assert np.array_equal(member[r].export(), o.rotate(y, s).data())
    assert np.array_equal(ctx.lintrans(x, "sigma", n, 4).export(), o.lt_sigma(y, n, 4).data())


def test_more_giant_steps_than_a_launch_takes(oracle_mod):
    """127 giant steps of sigma (one baby step, d = 64): 126 key inner products
    in two launches, the second onto the first; alone against the oracle, and
    in batches of three against each product alone"""
    from paper_2305_17341_amd import he
    n, ch, opts = 64, I.SMALL, {"n1_z": 1, "n1_t": 1}
    ctx = he.chain_context(ch, seed=80)
    ctx.keygen(ctx.matmul_rot_steps(n, opts))
    steps = he.lintrans_rot_steps("Z", n, 1)
    assert len(steps) == 126
    o = oracle_mod.Oracle(ch.log_n, ch.q_bits, ch.p_bits, seed=80)
    o.keygen(rot_steps=steps)
    A = I.uniform_matrix(5, n)
    g = ctx.lintrans(ctx.encrypt_matrix(A, nonce=2), "sigma", n, 1)
    w = o.lt_sigma(o.encrypt(A.ravel(), nonce=2), n, 1)
    assert g.level == w.level and g.scale == w.scale
    assert np.array_equal(g.export(), w.data())
    x = [ctx.encrypt_matrix(I.uniform_matrix(20 + i, n), nonce=20 + i) for i in range(6)]
    got = ctx.matmul_batch(x[:3], x[3:], [n] * 3, dict(opts, flags=BATCHED))
    for i in range(3):
        assert np.array_equal(got[i].export(), ctx.matmul(x[i], x[3 + i], n, opts).export()), i
