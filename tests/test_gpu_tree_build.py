"""GPU parity of tree_build (token-info sampling, Alg. 1, with budget pruning,
§5.2) against the CPU oracle, through the C ABI.

Tokens, parents and node counts must match bit for bit: every decision is
either a ranking of fp32 logit sums (identical on both sides) or a ranking of
fp64 joint probabilities, and the oracle reports how far apart the competing
joints were; the cases below are asserted to have margins far above the
fp64 rounding of either side. Joint probabilities (fp32 output) match to
1e-6 relative."""
import numpy as np
import pytest
import torch

from paper_2602_21224_amd import workloads as W
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def run_gpu(T, x, budget=None, k=None):
    budget = x.budget if budget is None else budget
    k = x.k if k is None else k
    H = x.H
    tab = U.dev(x.table.view(np.int16)).view(torch.bfloat16) if H > 0 else None
    par, tok, jnt, nn = T.tree_build(U.dev(x.logits), U.dev(x.root), tab,
                                     U.dev(x.hot_vocab) if H > 0 else None,
                                     U.dev(x.hot_index) if H > 0 else None, k=k, budget=budget)
    torch.cuda.synchronize()
    return par.cpu().numpy(), tok.cpu().numpy(), jnt.cpu().numpy(), nn.cpu().numpy()


def compare(oracle_mod, T, x, label, budget=None, k=None):
    budget = x.budget if budget is None else budget
    k = x.k if k is None else k
    print(f"case {label}: B={x.B} S={x.S} V={x.V} H={x.H} k={k} budget={budget}", flush=True)
    margins = []
    want = oracle_mod.tree_build(x.logits, x.root, x.table, x.hot_vocab, k, budget, margins)
    if margins:
        assert min(margins) > 1e-9, f"{label}: near-tie in the oracle ({min(margins):.2e})"
    got = run_gpu(T, x, budget, k)
    np.testing.assert_array_equal(got[3], want[3], err_msg=f"{label} num_nodes")
    np.testing.assert_array_equal(got[1], want[1], err_msg=f"{label} token")
    np.testing.assert_array_equal(got[0], want[0], err_msg=f"{label} parent")
    np.testing.assert_allclose(got[2], want[2], rtol=1e-6, atol=0, err_msg=f"{label} joint")
    return got


CASES = [
    # (B, S, V, H, k, budget)
    (1, 1, 10, 0, 1, 1),
    (2, 3, 300, 60, 3, 16),
    (3, 4, 1000, 1000, 4, 40),          # every token hot
    (2, 5, 777, 0, 5, 100),             # no token information at all
    (4, 2, 4096, 512, 16, 256),         # largest branch number and budget
    (2, 16, 600, 100, 2, 33),           # most steps
    (5, 7, 5000, 1200, 8, 64),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tree_build_cases(oracle_mod, case):
    T = U.require_gpu()
    B, S, V, H, k, budget = CASES[case]
    x = W.make_tree_build_inputs(f"c{case}", 100 + case, B=B, S=S, V=V, H=H, k=k, budget=budget)
    compare(oracle_mod, T, x, f"case{case}")


SPLITS = [
    # (B, S, V, H, k, budget): edges of the builder's splits
    (1, 2, 300000, 50, 3, 12),          # rows of more than one pass per segment
    (1, 2, 8200, 1025, 9, 40),          # more than 8 branches: one segment, one chunk;
    (17, 2, 8193, 2056, 8, 30),         # (8 branches: two unequal chunks)
    (9, 3, 70000, 32769, 10, 60),       # five segments, 17 chunks, rows not aligned;
    (3, 3, 4000, 4000, 16, 200),        # all hot, 16 branches
    (16, 2, 40000, 20001, 5, 20),       # odd hot count
    (64, 2, 8200, 2056, 3, 12),         # two segments of 16 tokens per thread, two chunks of 32 columns per lane
    (1, 2, 8200, 1025, 7, 40),          # five segments of 4 tokens per thread, two nearly empty chunks
    (3, 3, 4000, 4000, 8, 200),         # all hot, 8 branches
    (130, 2, 9000, 3000, 3, 12),        # more workgroups per step than run at once: separate launches
]


@pytest.mark.parametrize("case", range(len(SPLITS)))
def test_tree_build_splits(oracle_mod, case):
    T = U.require_gpu()
    B, S, V, H, k, budget = SPLITS[case]
    x = W.make_tree_build_inputs(f"s{case}", 130 + case, B=B, S=S, V=V, H=H, k=k, budget=budget)
    compare(oracle_mod, T, x, f"split{case}")


def test_tree_build_columns_in_passes(oracle_mod):
    """More hot tokens than 32 chunks of one pass hold (65536): every chunk runs
    in two passes whose winners and sums are merged. All table rows are the same
    row, so that the oracle needs only one of them."""
    T = U.require_gpu()
    B, S, V, H, k, budget = 1, 3, 70000, 66001, 4, 30
    print(f"case passes: V={V} H={H}", flush=True)
    x = W.make_tree_build_inputs("p", 140, B=B, S=S, V=V, H=64, k=k, budget=budget)
    rng = np.random.default_rng(1)
    hot = rng.permutation(V)[:H].astype(np.int32)
    index = np.full(V, -1, np.int32)
    index[hot] = np.arange(H, dtype=np.int32)
    row = W.f32_to_bf16_bits(rng.standard_normal(H, dtype=np.float32))
    margins = []
    want = oracle_mod.tree_build(x.logits, x.root, np.broadcast_to(row, (H, H)), hot, k, budget, margins)
    assert min(margins) > 1e-9
    tab = U.dev(row.view(np.int16)).view(torch.bfloat16).expand(H, H).contiguous()
    par, tok, jnt, nn = T.tree_build(U.dev(x.logits), U.dev(x.root), tab, U.dev(hot), U.dev(index),
                                     k=k, budget=budget)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tok.cpu().numpy(), want[1])
    np.testing.assert_array_equal(par.cpu().numpy(), want[0])
    np.testing.assert_allclose(jnt.cpu().numpy(), want[2], rtol=1e-6)


@pytest.mark.parametrize("H,k", [(0, 3), (3000, 8), (5000, 16), (3000, 11)])
def test_tree_build_equal_logits(H, k):
    """Every candidate ties: more than any candidate list holds, and the k lowest
    vocabulary ids win, with probability 1 / V each."""
    T = U.require_gpu()
    V, B, S = 5000, 2, 1
    rng = np.random.default_rng(H + k)
    hot = rng.permutation(V)[:H].astype(np.int32)
    index = np.full(V, -1, np.int32)
    index[hot] = np.arange(H, dtype=np.int32)
    logits = torch.full((B, S, V), -0.75, device="cuda")
    tab = torch.zeros((H, H), dtype=torch.bfloat16, device="cuda") if H else None
    roots = np.array([7, 4999], np.int32)
    par, tok, jnt, nn = T.tree_build(logits, U.dev(roots), tab, U.dev(hot) if H else None,
                                     U.dev(index) if H else None, k=k, budget=k + 1)
    torch.cuda.synchronize()
    for b in range(B):
        assert tok[b].tolist() == [int(roots[b])] + list(range(k))
        assert par[b].tolist() == [-1] + [0] * k
    np.testing.assert_allclose(jnt.cpu().numpy()[:, 1:], 1.0 / V, rtol=1e-6)
    assert (nn.cpu().numpy() == k + 1).all()


@pytest.mark.parametrize("mask", [-600.0, -1e4, -3.4028235e38])
@pytest.mark.parametrize("H,k", [(0, 8), (900, 8), (0, 12), (900, 3)])
def test_tree_build_masked_logits(oracle_mod, H, k, mask):
    """A constrained step: two allowed tokens, the others at one finite low value.
    Their probabilities underflow (to 0, or in products), so the budget beyond the
    live nodes goes to the nodes created first, as in the oracle. All its ties are
    exact on both sides, so no margin applies."""
    T = U.require_gpu()
    print(f"case masked H={H} k={k} mask={mask}", flush=True)
    x = W.make_tree_build_inputs("mask", 160 + k, B=3, S=4, V=2500, H=H, k=k, budget=64)
    if k == 3:                                             # hot ids in ascending order
        x.hot_vocab.sort()
        x.hot_index[x.hot_vocab] = np.arange(H, dtype=np.int32)
    rng = np.random.default_rng(k)
    logits = np.full_like(x.logits, mask)
    for b in range(x.B):
        for i in range(x.S):
            keep = rng.choice(x.V, 2, replace=False)
            logits[b, i, keep] = x.logits[b, i, keep]
    x.logits[:] = logits
    want = oracle_mod.tree_build(x.logits, x.root, x.table, x.hot_vocab, k, x.budget)
    got = run_gpu(T, x)
    np.testing.assert_array_equal(got[3], want[3])
    np.testing.assert_array_equal(got[1], want[1])
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_allclose(got[2], want[2], rtol=1e-6, atol=1e-45)


@pytest.mark.parametrize("V", [70000, 300000])
def test_tree_build_equal_logits_large(V):
    """The same ties with 16 tokens per thread, in one pass and in two."""
    T = U.require_gpu()
    k = 8
    logits = torch.full((1, 1, V), 2.0, device="cuda")
    par, tok, jnt, nn = T.tree_build(logits, U.dev(np.array([9], np.int32)), None, None, None, k=k, budget=k + 1)
    torch.cuda.synchronize()
    assert tok[0].tolist() == [9] + list(range(k))
    np.testing.assert_allclose(jnt[0, 1:].cpu().numpy(), 1.0 / V, rtol=1e-6)


def shared_row_inputs(seed, B, S, V, H, k, budget):
    """Inputs whose table rows are all the same row (so that a large table costs
    the oracle one row): the inputs and the bf16 table on the GPU."""
    x = W.make_tree_build_inputs("shared", seed, B=B, S=S, V=V, H=64, k=k, budget=budget)
    rng = np.random.default_rng(seed)
    x.hot_vocab = rng.permutation(V)[:H].astype(np.int32)
    x.hot_index = np.full(V, -1, np.int32)
    x.hot_index[x.hot_vocab] = np.arange(H, dtype=np.int32)
    row = W.f32_to_bf16_bits(rng.standard_normal(H, dtype=np.float32))
    x.table = np.broadcast_to(row, (H, H))
    x.root[0] = x.hot_vocab[5]
    return x, U.dev(row.view(np.int16)).view(torch.bfloat16).expand(H, H).contiguous()


def check_shared_row(oracle_mod, T, x, tab, alen=None):
    a = (U.dev(x.hot_vocab), U.dev(x.hot_index))
    margins = []
    if alen is None:
        want = oracle_mod.tree_build(x.logits, x.root, x.table, x.hot_vocab, x.k, x.budget, margins)
        got = T.tree_build(U.dev(x.logits), U.dev(x.root), tab, *a, k=x.k, budget=x.budget)
    else:
        want = oracle_mod.resample(x.logits, x.root, alen, x.table, x.hot_vocab, x.k, 1, x.budget, margins)
        got = T.tree_resample(U.dev(x.logits), U.dev(x.root), U.dev(alen), tab, *a, k=x.k, r=1,
                              budget=x.budget)
    torch.cuda.synchronize()
    assert min(margins) > 1e-9
    par, tok, jnt, nn = [t.cpu().numpy() for t in got]
    np.testing.assert_array_equal(nn, want[3])
    np.testing.assert_array_equal(tok, want[1])
    np.testing.assert_array_equal(par, want[0])
    np.testing.assert_allclose(jnt, want[2], rtol=1e-6)


@pytest.mark.parametrize("H,k,alen", [
    (28673, 8, None),          # 19 segments and 15 chunks of 8 keys: more than 4 keys per lane
    (28680, 5, [1, 2]),        # re-sampling, wide table loads
])
def test_tree_build_many_parts(oracle_mod, H, k, alen):
    """A vocabulary and hot set whose parts hold more than 256 candidate keys per
    node: the selection holds eight per lane."""
    T = U.require_gpu()
    print(f"case many parts H={H} k={k} accept_len={alen}", flush=True)
    B = len(alen) if alen else 1
    x, tab = shared_row_inputs(170 + k, B, 4 if alen else 3, 151936, H, k, 40)
    check_shared_row(oracle_mod, T, x, tab, None if alen is None else np.array(alen, np.int32))


def test_tree_build_many_parts_list_overflow(oracle_mod):
    """Every eighth part holds low values only: more keys reach the selection's
    first floor (the smallest of eight groups' maxima) than its list holds."""
    T = U.require_gpu()
    V, H, k = 151936, 43000, 8                 # 19 segments of 7997, 21 chunks of 2048
    print(f"case many parts overflow V={V} H={H} k={k}", flush=True)
    x, tab = shared_row_inputs(180, 1, 3, V, H, k, 40)
    seg = np.arange(V) // 7997
    low = (x.hot_index < 0) & (seg % 8 == 0)
    chunk = np.arange(H) // 2048
    low[x.hot_vocab[(19 + chunk) % 8 == 0]] = True
    x.logits[:, :, low] -= 60.0
    check_shared_row(oracle_mod, T, x, tab)


@pytest.mark.parametrize("B,S,V,H,k", [
    (9, 3, 70000, 32769, 6),   # 17 chunks of 32 columns per lane, rows not aligned
    (1, 3, 70000, 66048, 4),   # chunks of two passes, wide table loads in both
])
def test_tree_build_wide_chunks(oracle_mod, B, S, V, H, k):
    T = U.require_gpu()
    print(f"case wide chunks B={B} V={V} H={H} k={k}", flush=True)
    x, tab = shared_row_inputs(190 + k, B, S, V, H, k, 60)
    check_shared_row(oracle_mod, T, x, tab)


def test_tree_build_narrative(oracle_mod):
    """The worked example of §5.2 (golden fixture) on the GPU."""
    T = U.require_gpu()
    from tests.test_oracle_tree_build import narrative
    g, ids, logits, table, hot = narrative()
    V = len(g["vocab"])
    hot_index = np.arange(V, dtype=np.int32)
    x = W.TreeBuildInputs("narrative", 1, logits.shape[1], V, V, g["k"], 11, logits,
                          np.array([ids[g["root"]]], np.int32), table, hot, hot_index)
    par, tok, jnt, nn = compare(oracle_mod, T, x, "narrative")
    names = [g["vocab"][t] for t in tok[0]]
    assert names[3] == "server" and jnt[0, 3] == pytest.approx(0.42, rel=1e-6)
    assert names[7] == "optimization" and jnt[0, 7] == pytest.approx(0.294, rel=1e-6)


def test_tree_build_full_vocabulary(oracle_mod):
    """The 8B-shaped vocabulary (128256) with a quarter of the hot table (8192
    hot tokens)."""
    T = U.require_gpu()
    x = W.make_tree_build_inputs("full", 7, B=4, S=7, V=128256, H=8192, k=8, budget=64)
    compare(oracle_mod, T, x, "full-vocab")


def test_tree_build_and_resample_bench_presets(oracle_mod):
    """The benchmarked workloads themselves, whole: 16 sequences, 7 steps,
    vocabulary 128256 with 32768 hot tokens, k 8, budget 64; then re-sampling
    on the same inputs with the benchmark's accept lengths and bonus tokens."""
    T = U.require_gpu()
    x = W.tree_build_preset("tb_llama8b_bs16")
    compare(oracle_mod, T, x, "tb_llama8b_bs16")
    bonus, alen = W.resample_inputs(x, 7)
    compare_resample(oracle_mod, T, x, bonus, alen, 1, "rs_llama8b_bs16-shapes")


def test_tree_build_feeds_verification(oracle_mod):
    """The builder's (parent, token, num_nodes) are valid tree inputs of the
    verification calls: a ragged accept over them matches the oracle."""
    T = U.require_gpu()
    x = W.make_tree_build_inputs("feed", 9, B=3, S=3, V=500, H=100, k=3, budget=20)
    par, tok, jnt, nn = run_gpu(T, x)
    assert (nn == 1 + 3 + 2 * 9).all() or (nn == 20).all()
    rng = np.random.default_rng(0)
    logits = rng.standard_normal((x.B, x.budget, x.V)).astype(np.float32)
    a, alen, aidx, bonus = T.tree_argmax_accept(U.dev(logits), U.dev(tok), U.dev(par),
                                                num_nodes=U.dev(nn))
    torch.cuda.synchronize()
    ra = oracle_mod.argmax(logits)
    rl, ri, rb = oracle_mod.accept(tok, par, ra, num_nodes=nn)
    np.testing.assert_array_equal(alen.cpu().numpy(), rl)
    np.testing.assert_array_equal(aidx.cpu().numpy(), ri)
    np.testing.assert_array_equal(bonus.cpu().numpy(), rb)


def test_tree_build_reuses_workspace(oracle_mod):
    """Two calls in a row on one workspace, the second smaller: nothing of the
    first call leaks into the second."""
    T = U.require_gpu()
    big = W.make_tree_build_inputs("big", 21, B=4, S=6, V=3000, H=700, k=6, budget=80)
    small = W.make_tree_build_inputs("small", 22, B=2, S=2, V=400, H=50, k=2, budget=9)
    ws = torch.empty(T.tree_build_workspace_size(4, 6, 3000, 700, 6), dtype=torch.uint8,
                     device="cuda")
    for x in (big, small):
        tab = U.dev(x.table.view(np.int16)).view(torch.bfloat16)
        par, tok, jnt, nn = T.tree_build(U.dev(x.logits), U.dev(x.root), tab, U.dev(x.hot_vocab),
                                         U.dev(x.hot_index), k=x.k, budget=x.budget, workspace=ws)
        torch.cuda.synchronize()
        want = oracle_mod.tree_build(x.logits, x.root, x.table, x.hot_vocab, x.k, x.budget)
        np.testing.assert_array_equal(tok.cpu().numpy(), want[1])
        np.testing.assert_array_equal(par.cpu().numpy(), want[0])
        np.testing.assert_array_equal(nn.cpu().numpy(), want[3])


@pytest.mark.parametrize("k", [4, 12])
def test_tree_build_workspace_alignment(oracle_mod, k):
    """The expansions load several columns per lane at once where the table (and,
    in separate launches, as more than 8 branches take, the hot ids and the
    workspace row) are aligned for it; a workspace that is only 8-byte aligned (the
    documented minimum), or a table and hot-id array one element off, take the
    narrow loads and build the same trees."""
    T = U.require_gpu()
    x = W.make_tree_build_inputs("align", 23, B=2, S=3, V=5000, H=4096, k=k, budget=30)
    n = T.tree_build_workspace_size(x.B, x.S, x.V, x.H, x.k)
    ws = torch.empty(n + 16, dtype=torch.uint8, device="cuda")
    margins = []
    want = oracle_mod.tree_build(x.logits, x.root, x.table, x.hot_vocab, x.k, x.budget, margins)
    assert min(margins) > 1e-9
    tab = U.dev(x.table.view(np.int16)).view(torch.bfloat16)
    got = []
    for off in (0, 8):
        print(f"case workspace offset {off}", flush=True)
        par, tok, jnt, nn = T.tree_build(U.dev(x.logits), U.dev(x.root), tab, U.dev(x.hot_vocab),
                                         U.dev(x.hot_index), k=x.k, budget=x.budget,
                                         workspace=ws[off:off + n])
        torch.cuda.synchronize()
        got.append((par.cpu().numpy(), tok.cpu().numpy(), jnt.cpu().numpy(), nn.cpu().numpy()))
        np.testing.assert_array_equal(got[-1][3], want[3])
        np.testing.assert_array_equal(got[-1][1], want[1])
        np.testing.assert_array_equal(got[-1][0], want[0])
        np.testing.assert_allclose(got[-1][2], want[2], rtol=1e-6, atol=0)
    for a, b in zip(got[0][:2] + got[0][3:], got[1][:2] + got[1][3:]):
        np.testing.assert_array_equal(a, b)
    # the caller's table and hot ids off the wide loads' alignment (one element
    # into a larger buffer): the narrow loads, the same trees
    print("case table and hot ids one element off", flush=True)
    tbuf = torch.empty(x.H * x.H + 1, dtype=torch.bfloat16, device="cuda")
    tbuf[1:].copy_(tab.reshape(-1))
    vbuf = torch.empty(x.H + 1, dtype=torch.int32, device="cuda")
    vbuf[1:].copy_(U.dev(x.hot_vocab))
    par, tok, jnt, nn = T.tree_build(U.dev(x.logits), U.dev(x.root), tbuf[1:].view(x.H, x.H),
                                     vbuf[1:], U.dev(x.hot_index), k=x.k, budget=x.budget,
                                     workspace=ws[:n])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(nn.cpu().numpy(), want[3])
    np.testing.assert_array_equal(tok.cpu().numpy(), want[1])
    np.testing.assert_array_equal(par.cpu().numpy(), want[0])
    np.testing.assert_allclose(jnt.cpu().numpy(), want[2], rtol=1e-6, atol=0)


@pytest.mark.parametrize("k", [4, 8, 12])
@pytest.mark.parametrize("H", [0, 600])
def test_tree_build_not_finite_stays_in_bounds(H, k):
    """Logits and table entries that are not finite break the contract, so the
    tree is unspecified, but NaN joint probabilities must not leave frontier slots
    or kept nodes undefined: node counts and links stay valid, and nothing is
    written outside the outputs."""
    T = U.require_gpu()
    B, S, V, budget, pad = 5, 4, 3000, 20, 64
    print(f"case not finite H={H} k={k}", flush=True)
    x = W.make_tree_build_inputs("nf", 150 + k, B=B, S=S, V=V, H=H, k=k, budget=budget)
    logits = x.logits.copy()
    rng = np.random.default_rng(k)
    logits[0] = np.nan                                     # no candidate at all
    logits[1][rng.random((S, V)) < 0.3] = np.nan
    logits[2, :, rng.integers(0, V, 3)] = np.inf
    logits[3] = -np.inf                                    # fewer candidates than branches, then infinities
    logits[3, 0, 17] = 1.0
    logits[3, 1:, :] = np.inf
    tab = None
    if H:
        bits = x.table.copy()
        bits[::3, ::5] = 0x7FC0                            # NaN
        bits[1::3, ::7] = 0x7F80                           # +inf
        tab = U.dev(bits.view(np.int16)).view(torch.bfloat16)
    buf = {n: torch.full((2 * pad + B * budget,), 7, dtype=dt, device="cuda")
           for n, dt in (("parent", torch.int32), ("token", torch.int32), ("joint", torch.float32))}
    out = {n: t[pad:-pad].view(B, budget) for n, t in buf.items()}
    par, tok, jnt, nn = T.tree_build(U.dev(logits), U.dev(x.root), tab, U.dev(x.hot_vocab) if H else None,
                                     U.dev(x.hot_index) if H else None, k=k, budget=budget, **out)
    torch.cuda.synchronize()
    for n, t in buf.items():
        assert (t[:pad] == 7).all() and (t[-pad:] == 7).all(), f"{n}: written outside"
    assert (nn == budget).all()
    par, tok = par.cpu().numpy(), tok.cpu().numpy()
    assert (par >= -1).all() and (par < np.arange(budget)).all()
    assert (tok >= -1).all() and (tok < V).all()


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("H,k", [(0, 3), (3000, 8), (3000, 12)])
def test_tree_build_nan_is_no_candidate(H, k, ties):
    """Beside finite candidates NaN logits are left out of the tree and of the
    sums, whichever way the candidates are ranked: a few lie above the others, or
    (ties) more are equal than any candidate list holds."""
    T = U.require_gpu()
    print(f"case nan H={H} k={k} ties={ties}", flush=True)
    V, B = 5000, 2
    rng = np.random.default_rng(H + k)
    hot = rng.permutation(V)[:H].astype(np.int32)
    index = np.full(V, -1, np.int32)
    index[hot] = np.arange(H, dtype=np.int32)
    logits = np.full((B, 1, V), 0.5, np.float32)
    if not ties:
        logits += rng.random((B, 1, V), dtype=np.float32)
    nan = rng.random((B, 1, V)) < 0.2
    logits[nan] = np.nan
    tab = torch.zeros((H, H), dtype=torch.bfloat16, device="cuda") if H else None
    par, tok, jnt, nn = T.tree_build(U.dev(logits), U.dev(np.array([7, 4999], np.int32)), tab,
                                     U.dev(hot) if H else None, U.dev(index) if H else None, k=k, budget=k + 1)
    torch.cuda.synchronize()
    for b in range(B):
        x = np.where(nan[b, 0], -np.inf, logits[b, 0].astype(np.float64))
        order = np.lexsort((np.arange(V), -x))[:k]
        assert tok[b, 1:].tolist() == order.tolist()
        p = np.exp(x[order] - x.max()) / np.exp(x - x.max()).sum()
        np.testing.assert_allclose(jnt[b, 1:].cpu().numpy(), p, rtol=1e-6)


# ---------------------------------------------------------------- re-sampling (Alg. 2)
def run_resample(T, x, bonus, alen, r, budget=None, k=None):
    budget = x.budget if budget is None else budget
    k = x.k if k is None else k
    H = x.H
    tab = U.dev(x.table.view(np.int16)).view(torch.bfloat16) if H > 0 else None
    out = T.tree_resample(U.dev(x.logits), U.dev(bonus), U.dev(alen), tab,
                          U.dev(x.hot_vocab) if H > 0 else None,
                          U.dev(x.hot_index) if H > 0 else None, k=k, r=r, budget=budget)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


def compare_resample(oracle_mod, T, x, bonus, alen, r, label):
    print(f"case {label}: B={x.B} S={x.S} V={x.V} H={x.H} k={x.k} r={r} "
          f"accept_len={alen.tolist()}", flush=True)
    margins = []
    want = oracle_mod.resample(x.logits, bonus, alen, x.table, x.hot_vocab, x.k, r, x.budget,
                               margins)
    if margins:
        assert min(margins) > 1e-9, f"{label}: near-tie in the oracle ({min(margins):.2e})"
    got = run_resample(T, x, bonus, alen, r)
    np.testing.assert_array_equal(got[3], want[3], err_msg=f"{label} num_nodes")
    np.testing.assert_array_equal(got[1], want[1], err_msg=f"{label} token")
    np.testing.assert_array_equal(got[0], want[0], err_msg=f"{label} parent")
    np.testing.assert_allclose(got[2], want[2], rtol=1e-6, atol=0, err_msg=f"{label} joint")
    return got


@pytest.mark.parametrize("case", range(6))
def test_resample_cases(oracle_mod, case):
    """The fourth and fifth in separate launches (more than 8 branches); the last a
    batch that a first tree would take to them."""
    T = U.require_gpu()
    B, S, V, H, k, budget, r = [(6, 5, 800, 200, 3, 30, 1), (8, 7, 5000, 1000, 8, 64, 2),
                                (4, 16, 600, 0, 2, 40, 0), (6, 5, 3000, 800, 12, 60, 1),
                                (5, 6, 900, 0, 9, 30, 0), (130, 4, 9000, 3000, 3, 20, 1)][case]
    x = W.make_tree_build_inputs(f"rs{case}", 200 + case, B=B, S=S, V=V, H=H, k=k, budget=budget)
    rng = np.random.default_rng(case)
    alen = rng.integers(0, S + 2, B).astype(np.int32)         # 0 .. S+1, every window kind
    alen[0], alen[-1] = 1, S + 1
    bonus = rng.integers(0, V, B).astype(np.int32)
    if H:
        bonus[1::2] = x.hot_vocab[rng.integers(0, H, len(bonus[1::2]))]
    compare_resample(oracle_mod, T, x, bonus, alen, r, f"resample{case}")


def test_resample_narrative(oracle_mod):
    """The re-sampling narrative of §5.3 (golden fixture) on the GPU."""
    T = U.require_gpu()
    from tests.test_oracle_tree_build import resample_narrative
    g, ids, logits, table, hot = resample_narrative()
    V = len(g["vocab"])
    x = W.TreeBuildInputs("rs-narrative", 1, logits.shape[1], V, V, g["k"], 16, logits,
                          np.array([0], np.int32), table, hot, np.arange(V, dtype=np.int32))
    got = compare_resample(oracle_mod, T, x, np.array([ids[g["bonus"]]], np.int32),
                           np.array([g["accept_len"]], np.int32), g["r"], "rs-narrative")
    names = [g["vocab"][t] for t in got[1][0][:3]]
    assert names == ["quantization", "accuracy", "method"]


def test_speculative_iteration_chain(oracle_mod):
    """One speculative iteration end to end on the GPU, each stage checked
    against the oracle: build the draft trees, verify them (greedy accept over
    synthetic target logits with some drafts made acceptable), re-sample from
    the bonus tokens and accepted lengths."""
    T = U.require_gpu()
    x = W.make_tree_build_inputs("chain", 77, B=6, S=5, V=2000, H=400, k=3, budget=24)
    par, tok, jnt, nn = run_gpu(T, x)
    want = oracle_mod.tree_build(x.logits, x.root, x.table, x.hot_vocab, x.k, x.budget)
    np.testing.assert_array_equal(tok, want[1])
    rng = np.random.default_rng(3)
    tgt = rng.standard_normal((x.B, x.budget, x.V)).astype(np.float32)
    for b in range(x.B):                                   # let the target agree on a path
        depth = int(rng.integers(0, 4))
        i = 0
        for _ in range(depth):
            kids = [c for c in range(1, nn[b]) if par[b, c] == i]
            if not kids:
                break
            c = kids[int(rng.integers(0, len(kids)))]
            tgt[b, i, tok[b, c]] += 50.0
            i = c
    a, alen, aidx, bonus = T.tree_argmax_accept(U.dev(tgt), U.dev(tok), U.dev(par),
                                                num_nodes=U.dev(nn))
    torch.cuda.synchronize()
    alen, bonus = alen.cpu().numpy(), bonus.cpu().numpy()
    rl, ri, rb = oracle_mod.accept(tok, par, oracle_mod.argmax(tgt), num_nodes=nn)
    np.testing.assert_array_equal(alen, rl)
    np.testing.assert_array_equal(bonus, rb)
    print(f"accept_len {alen.tolist()}", flush=True)
    compare_resample(oracle_mod, T, x, bonus, alen, 1, "chain-resample")
