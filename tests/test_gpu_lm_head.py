"""GPU parity of tree_lm_head_argmax_accept (the LM head fused with greedy
verification) against the CPU oracle, through the C ABI.

The kernel sums bf16 products in fp32 on the matrix cores, the oracle sums
them exactly (fp64). Any fp32 summation order puts a computed logit within
gamma_d * sum_i |h_i w_vi| of the exact one (gamma_d = d u / (1 - d u),
u = 2^-24; the products themselves are exact in fp32), and
sum_i |h_i w_vi| <= sum_i |h_i| * max|W| =: S_r for every v. So:
  * rows whose exact top-2 margin exceeds 2 gamma_d S_r have one correct
    answer and must match the oracle's argmax exactly;
  * on the other rows several entries are correct fp32 argmaxes: the GPU's
    pick must be a valid vocabulary id whose exact logit lies within
    2 gamma_d S_r of the exact maximum.
Acceptance (accept_len, accept_idx, bonus) is checked bit-exactly against the
oracle's acceptance applied to the argmax the GPU produced."""
import numpy as np
import pytest
import torch

from paper_2602_21224_amd import workloads as W
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def gamma(d):
    u = 2.0 ** -24
    return d * u / (1 - d * u)


def upload(x):
    return (U.dev_bf16(x.hidden), U.dev_bf16(x.w_head), U.dev(x.draft), U.dev(x.parent),
            None if x.num_nodes is None else U.dev(x.num_nodes))


def run_gpu(T, x, ws=None):
    hid, w, draft, par, nn = upload(x)
    out = T.tree_lm_head_argmax_accept(hid, w, draft, par, num_nodes=nn, workspace=ws)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


def real_rows(x):
    counts = np.full(x.B, x.N) if x.num_nodes is None else np.clip(x.num_nodes, 0, x.N)
    return np.array([b * x.N + i for b in range(x.B) for i in range(int(counts[b]))], np.int64)


def check_argmax(oracle_mod, x, got_amax, rows, label, min_decisive=0.5):
    """Check the GPU's argmax of the given flat rows (see the module docstring)."""
    hid = x.hidden.reshape(-1, x.d)[rows]
    got = got_amax.reshape(-1)[rows]
    want, margin, _ = oracle_mod.lm_head_argmax(hid, x.w_head)
    h = W.bf16_bits_to_f32(hid).astype(np.float64)
    wmax = float(np.abs(W.bf16_bits_to_f32(x.w_head)).max())
    bound = gamma(x.d) * np.abs(h).sum(1) * wmax
    decisive = margin > 2 * bound
    print(f"[{label}] {len(rows)} rows, {decisive.sum()} decisive", flush=True)
    assert decisive.mean() >= min_decisive, f"{label}: too few decisive rows for a parity check"
    np.testing.assert_array_equal(got[decisive], want[decisive], err_msg=f"{label} argmax")
    assert ((got >= 0) & (got < x.V)).all(), f"{label}: argmax out of range"
    for j in np.nonzero(~decisive)[0]:
        wg = W.bf16_bits_to_f32(x.w_head[got[j]]).astype(np.float64)
        ww = W.bf16_bits_to_f32(x.w_head[want[j]]).astype(np.float64)
        assert h[j] @ wg >= h[j] @ ww - 2 * bound[j], f"{label}: row {rows[j]} picked a non-maximum"


def check_accept(oracle_mod, x, got, label):
    amax, alen, aidx, bonus = got
    padding = np.ones(x.B * x.N, bool)
    padding[real_rows(x)] = False
    assert (amax.reshape(-1)[padding] == -1).all(), f"{label}: padding rows got an argmax"
    rl, ri, rb = oracle_mod.accept(x.draft, x.parent, amax, num_nodes=x.num_nodes)
    np.testing.assert_array_equal(alen, rl, err_msg=f"{label} accept_len")
    np.testing.assert_array_equal(aidx, ri, err_msg=f"{label} accept_idx")
    np.testing.assert_array_equal(bonus, rb, err_msg=f"{label} bonus")


CASES = [
    # (B, N, V, d, num_nodes)
    (2, 16, 1000, 256, None),
    (3, 37, 1000, 192, [37, 5, 20]),     # ragged rows and vocabulary, three K units
    (1, 8, 257, 64, None),               # one K unit, one entry past a vocabulary tile
    (2, 4, 300, 128, None),              # two K units
    (1, 3, 1, 128, None),                # a single vocabulary entry
    (4, 64, 20000, 1024, None),          # full row tile, many vocabulary tiles
    (5, 64, 3000, 512, [64, 0, 17, 64, 1]),   # row tiles split across sequences, empty ones
    (6, 64, 900, 320, None),             # two row blocks, five K units: a rotated group of four + one
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_lm_head_cases(oracle_mod, case):
    T = U.require_gpu()
    B, N, V, d, nn = CASES[case]
    print(f"case lm{case}: B={B} N={N} V={V} d={d} num_nodes={nn}", flush=True)
    x = W.make_lm_head_inputs(f"lm{case}", 300 + case, B=B, N=N, V=V, d=d, num_nodes=nn)
    got = run_gpu(T, x)
    rows = real_rows(x)
    if len(rows):
        check_argmax(oracle_mod, x, got[0], rows, f"lm{case}",
                     min_decisive=0.0 if V == 1 else 0.5)
    check_accept(oracle_mod, x, got, f"lm{case}")


FEW_ROWS = [
    # (B, N, V, d): every split of the weight stream (up to 128 rows) at its edges
    (1, 1, 5, 64),             # one row, one unit, a vocabulary shorter than a wave's rows
    (1, 16, 257, 128),         # ranges of 15 and 16 rows
    (1, 17, 1000, 192),
    (1, 24, 24600, 2048),      # two 4-wave workgroups per CU: up to 32 rows,
    (1, 33, 24577, 2048),      # up to 64
    (1, 32, 40961, 128),       # two 8-wave workgroups per CU: up to 32 rows,
    (2, 20, 41000, 64),        # up to 64; a range's second tile has idle waves
    (3, 8, 99999, 128),        # 32 rows per wave, up to 32 rows,
    (1, 64, 98305, 64),        # up to 64
    (1, 65, 3000, 320),        # more than 64 rows: the smallest and the largest
    (2, 64, 98400, 64),
    (3, 43, 2000, 128),        # 129 rows: the tiled product
    (10, 60, 25700, 64),       # three row blocks, more tiles than workgroups: the block changes per tile
    (5, 60, 33100, 192),       # two row blocks: a workgroup keeps its block over its tiles
]


@pytest.mark.parametrize("case", range(len(FEW_ROWS)))
def test_lm_head_few_rows(oracle_mod, case):
    """The same bound as the other cases (any fp32 summation order)."""
    T = U.require_gpu()
    B, N, V, d = FEW_ROWS[case]
    print(f"case lm few rows {case}: B={B} N={N} V={V} d={d}", flush=True)
    x = W.make_lm_head_inputs(f"few{case}", 330 + case, B=B, N=N, V=V, d=d)
    got = run_gpu(T, x)
    check_argmax(oracle_mod, x, got[0], real_rows(x), f"few{case}")
    check_accept(oracle_mod, x, got, f"few{case}")


def test_lm_head_full_size_row_block(oracle_mod):
    """The 8B-shaped head (vocabulary 128256, hidden size 4096, 16 x 64 nodes)
    in the launch configuration the benchmark times; the oracle checks one
    complete 256-row tile block (rows 512..767, sequences 8..11) over the whole
    vocabulary, the acceptance all 1024 rows."""
    T = U.require_gpu()
    print("case lm_llama8b_bs16 (row block 2 of 4)", flush=True)
    x = W.lm_head_preset("lm_llama8b_bs16")
    got = run_gpu(T, x)
    rows = np.arange(512, 768)
    check_argmax(oracle_mod, x, got[0], rows, "lm_llama8b_bs16")
    check_accept(oracle_mod, x, got, "lm_llama8b_bs16")
    assert (got[1] > 1).sum() >= 4, "planted drafts should be accepted somewhere"


def test_lm_head_equal_rows_pick_lowest_id(oracle_mod):
    """Two identical head rows give bit-identical sums (same operands, same
    accumulation order), so the lower id must win, as in the definition."""
    T = U.require_gpu()
    x = W.make_lm_head_inputs("ties", 310, B=2, N=16, V=3000, d=512)
    want, _, _ = oracle_mod.lm_head_argmax(x.hidden.reshape(-1, x.d), x.w_head)
    r = 3
    win = int(want[r])
    low = 7 if win != 7 else 8
    x.w_head[low] = x.w_head[win]          # an earlier duplicate of row r's winner
    got = run_gpu(T, x)
    assert got[0].reshape(-1)[r] == min(low, win)


@pytest.mark.parametrize("B", [1, 4])
def test_lm_head_equal_rows_everywhere(B):
    """The same for duplicates in every place that a kernel compares two values:
    64 rows take the weight's stream, 256 the tiled product. A hidden row is the
    head row it ties on (so that its logit there is the maximum by far), and the
    copy lies further on by: a value of the same lane, a lane of the other half,
    another 16- or 32-row block, another wave, another workgroup, another tile of
    the same workgroup. The last row's maximum is the last entry of a vocabulary
    that is no multiple of a tile."""
    T = U.require_gpu()
    V, d, N = 76777, 64, 64                # 300 tiles of 256: workgroups 0..43 have two
    print(f"case ties everywhere B={B} V={V}", flush=True)
    rng = np.random.default_rng(B)
    w = W.f32_to_bf16_bits(rng.standard_normal((V, d), dtype=np.float32))
    h = W.f32_to_bf16_bits(rng.standard_normal((B * N, d), dtype=np.float32))
    offs = (1, 2, 4, 8, 16, 32, 64, 128, 256, 300, 2048, 65536)
    want = {}
    for i, off in enumerate(offs):
        for rep in range(4):               # in different rows of the block and of the tile
            r = (i * 4 + rep) * B + rep % B
            v = 256 * (i * 3 % 40) + 61 * rep + 5 * i
            w[v + off] = w[v]
            h[r] = w[v]
            want[r] = v
    last = B * N - 1
    h[last] = w[V - 1]
    want[last] = V - 1
    rows = np.array(list(want))
    assert len(rows) == 4 * len(offs) + 1
    par = np.tile(np.arange(-1, N - 1, dtype=np.int32), (B, 1))
    am, *_ = T.tree_lm_head_argmax_accept(U.dev_bf16(h.reshape(B, N, d)), U.dev_bf16(w),
                                          U.dev(np.zeros((B, N), np.int32)), U.dev(par))
    torch.cuda.synchronize()
    exact = W.bf16_bits_to_f32(h[rows]).astype(np.float64) @ W.bf16_bits_to_f32(w).astype(np.float64).T
    np.testing.assert_array_equal(exact.argmax(1), list(want.values()))
    np.testing.assert_array_equal(am.cpu().numpy().reshape(-1)[rows], list(want.values()))


def test_lm_head_longest_rows_in_blocks():
    """A hidden size from 2^23 on takes the weight's stream for any number of
    rows, 128 rows per launch. Every hidden row is a head row, whose logit is
    above the others' by a factor of about sqrt(d)."""
    T = U.require_gpu()
    B, N, V, d = 3, 100, 200, 1 << 23
    print(f"case longest rows R={B * N} V={V} d={d}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    w = torch.randn((V, d), generator=g, device="cuda", dtype=torch.bfloat16)
    pick = torch.randint(0, V, (B * N,), generator=g, device="cuda")
    h = w[pick].view(B, N, d)
    par = torch.arange(-1, N - 1, device="cuda", dtype=torch.int32).repeat(B, 1).contiguous()
    am, *_ = T.tree_lm_head_argmax_accept(h, w, torch.zeros((B, N), dtype=torch.int32, device="cuda"), par)
    torch.cuda.synchronize()
    assert am.reshape(-1).tolist() == pick.tolist()


def test_lm_head_tiled_special_values(oracle_mod):
    """The tiled product's search for the lowest entry of the maximum: a hidden
    row of zeros ties every entry at 0 (entry 0 wins), two infinite logits tie
    at +inf (the lower one wins), a NaN entry beats both, and other rows are
    untouched by their neighbours."""
    T = U.require_gpu()
    x = W.make_lm_head_inputs("special", 312, B=4, N=64, V=3000, d=128)
    h = x.hidden.reshape(-1, x.d)
    h[7] = 0
    h[200] = 0
    h[200, 5] = W.f32_to_bf16_bits(np.array([1.0], np.float32))[0]
    x.w_head[1500, 5] = x.w_head[2900, 5] = 0x7F80            # +inf
    keep = np.delete(np.arange(256), [7, 200])
    h[keep, 5] = 0x8000                                       # -0 * inf = NaN
    got = run_gpu(T, x)[0].reshape(-1)
    assert got[7] == 1500 and got[200] == 1500                # 0 * inf = NaN; 1 * inf = inf
    assert (got[keep] == 1500).all()
    x.w_head[1500, 5] = x.w_head[2900, 5] = 0
    h[keep, 5] = 0
    got = run_gpu(T, x)[0]
    assert got.reshape(-1)[7] == 0
    check_argmax(oracle_mod, x, got, keep, "special")


def test_lm_head_nan_column_wins():
    """A NaN anywhere in head row v makes every logit of column v NaN, and NaN
    counts as the maximum (first NaN on ties), so every node's argmax is v."""
    T = U.require_gpu()
    x = W.make_lm_head_inputs("nan", 311, B=2, N=8, V=700, d=128)
    x.w_head[600, 17] = W.BF16_NAN
    x.w_head[650, 3] = W.BF16_NAN
    got = run_gpu(T, x)
    assert (got[0] == 600).all()


def test_lm_head_reuses_workspace(oracle_mod):
    """Two calls in a row on one workspace, the second smaller: the row keys
    are reset by each call."""
    T = U.require_gpu()
    big = W.make_lm_head_inputs("big", 312, B=4, N=64, V=2000, d=256)
    small = W.make_lm_head_inputs("small", 313, B=1, N=10, V=500, d=64)
    ws = torch.empty(T.lm_head_workspace_size(4, 64, 2000, 256), dtype=torch.uint8, device="cuda")
    for x in (big, small):
        got = run_gpu(T, x, ws)
        check_argmax(oracle_mod, x, got[0], real_rows(x), x.name)
        check_accept(oracle_mod, x, got, x.name)


def test_lm_head_matches_unfused_path(oracle_mod):
    """Fused and unfused verification agree: logits computed by torch (bf16
    inputs, fp32 result) fed to tree_argmax_accept give the same acceptance
    wherever the rows are decisive."""
    T = U.require_gpu()
    x = W.make_lm_head_inputs("unfused", 314, B=4, N=64, V=5000, d=1024)
    hid, w, draft, par, _ = upload(x)
    fused = T.tree_lm_head_argmax_accept(hid, w, draft, par)
    logits = (hid.float().reshape(-1, x.d) @ w.float().t().contiguous()).reshape(x.B, x.N, x.V)
    unfused = T.tree_argmax_accept(logits.contiguous(), draft, par)
    torch.cuda.synchronize()
    want, margin, _ = oracle_mod.lm_head_argmax(x.hidden.reshape(-1, x.d), x.w_head)
    h = W.bf16_bits_to_f32(x.hidden.reshape(-1, x.d)).astype(np.float64)
    bound = gamma(x.d) * np.abs(h).sum(1) * float(np.abs(W.bf16_bits_to_f32(x.w_head)).max())
    dec = margin > 2 * bound
    fa, ua = fused[0].cpu().numpy().reshape(-1), unfused[0].cpu().numpy().reshape(-1)
    np.testing.assert_array_equal(fa[dec], ua[dec])
    np.testing.assert_array_equal(fa[dec], want[dec])
