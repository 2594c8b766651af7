"""Parity with the fp64 oracle where the single-launch kernel changes its form: batches of one to
eight rows (rows of 16 KB down to 1 KB, full and partly filled segments), ragged ends of every
batch, one ranking or another by the number of candidates and of k, and more groups than a wave
has lanes.  Tolerances are those of test_gpu_parity.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from coral_inputs import Head, HeadConfig, make_hidden, to_storage  # noqa: E402
from oracle import compare  # noqa: E402
from test_gpu_parity import (TIGHT_LOGIT_ERR, TIGHT_LOGP_ERR, DeviceHead, check_dense, check_grouped, check_logprob, coral, run_dense,  # noqa: E402,F401
                             run_grouped, run_logprob)


def ragged_head(cfg, sizes, bias_std=0.5):
    rng = np.random.default_rng(cfg.seed)
    V = int(sum(sizes))
    perm = rng.permutation(V).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    rows = np.concatenate([np.sort(perm[offsets[n]:offsets[n + 1]]) for n in range(len(sizes))]).astype(np.int32)
    lm_W = to_storage(rng.standard_normal((V, cfg.H), dtype=np.float32) * np.float32(0.02), cfg.dtype)
    gate_W = to_storage(rng.standard_normal((len(sizes), cfg.H), dtype=np.float32) * np.float32(0.02), cfg.dtype)
    bias = (rng.standard_normal(len(sizes)) * bias_std).astype(np.float32)
    return Head(cfg, lm_W, gate_W, bias, offsets, rows)


def check_all(coral, cfg, sizes, Ms, dense=True):
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    for M in Ms:
        hidden = make_hidden(cfg, M, M)
        print(f"case {cfg.name} {cfg.dtype} H={cfg.H} M={M} G={cfg.G} g={cfg.g} k={cfg.k}", flush=True)
        check_grouped(dh, hidden, cfg.g, cfg.k, run_grouped(coral, dh, hidden, cfg.g, cfg.k))
        out = run_logprob(coral, dh, hidden, cfg.g, cfg.k)
        check_logprob(dh, hidden, cfg.g, cfg.k, out)
        again = run_logprob(coral, dh, hidden, cfg.g, cfg.k)
        assert all(np.array_equal(x, y) for x, y in zip(out, again))
        if dense:
            check_dense(dh, hidden, cfg.k, run_dense(coral, dh, hidden, cfg.k))


# (storage, H): segments per row 1, 2 | 3, 4 | 5, 8 | 10 (one value short of and past), 13, 16
WIDTHS = [("bf16", 512), ("f16", 1016), ("bf16", 1032), ("f32", 1024), ("f16", 2056), ("f32", 2048),
          ("bf16", 4616), ("f16", 5120), ("f32", 2564), ("bf16", 6664), ("f32", 4096), ("bf16", 8192)]


@pytest.mark.parametrize("dtype,H", WIDTHS)
def test_row_widths_and_ragged_batches(coral, dtype, H):
    sizes = [1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 64, 65, 127, 250]
    cfg = HeadConfig(f"width{H}", dtype, H, sum(sizes), len(sizes), 5, (1,), 9, 700 + H, True)
    check_all(coral, cfg, sizes, (1, 2, 3, 5, 8))


@pytest.mark.parametrize("k", [16, 17, 32, 33, 64])
@pytest.mark.parametrize("H,M", [(256, 1), (256, 9), (3072, 2)])
def test_many_candidates(coral, k, H, M):
    """k beyond what a sample of 64 lanes bounds, lists of one to a few rows per workgroup."""
    sizes = [40 + 13 * n for n in range(12)]
    cfg = HeadConfig(f"k{k}", "bf16", H, sum(sizes), 12, 3, (M,), k, 800 + k + H, True)
    check_all(coral, cfg, sizes, (M,))


@pytest.mark.parametrize("k", [10, 64])
def test_candidates_beyond_the_collecting_buffers(coral, k):
    """About 1200 rows per (workgroup, token): sorted lists per wave instead of buffers."""
    cfg = HeadConfig(f"lists{k}", "bf16", 64, 300_000, 2, 2, (3,), k, 820 + k, True)
    check_all(coral, cfg, [140_000, 160_000], (3,))


@pytest.mark.parametrize("G,g", [(64, 64), (65, 4), (128, 64), (129, 65), (300, 7), (1024, 16), (1024, 70)])
def test_many_groups(coral, G, g):
    sizes = [2 + (5 * n) % 7 for n in range(G)]
    cfg = HeadConfig(f"groups{G}", "f32", 128, sum(sizes), G, g, (1,), min(8, g), 840 + G + g, True)
    check_all(coral, cfg, sizes, (1, 3, 18), dense=False)


def test_equal_logits_in_the_single_launch_kernel(coral):
    """All-zero hidden vectors: every bound ties, the lower ids win."""
    sizes = [900, 1100, 1000]
    for k in (5, 64):
        cfg = HeadConfig("zero", "bf16", 512, sum(sizes), 3, 2, (2,), k, 860, True)
        dh = DeviceHead(coral, ragged_head(cfg, sizes))
        hidden = np.zeros((2, 512), np.uint16)
        check_grouped(dh, hidden, 2, k, run_grouped(coral, dh, hidden, 2, k))
        check_dense(dh, hidden, k, run_dense(coral, dh, hidden, k))


# The general path's tile kernels: widths that leave the last 512-column (fp32: 256-column) chunk
# partly filled, by one 16-byte vector up to one short of whole; one to four token tiles; fp32.
GENERAL = [("bf16", 4104, 9), ("f16", 4160, 8), ("bf16", 5112, 33), ("bf16", 520, 64), ("f16", 1000, 50),
           ("f32", 2052, 20), ("f32", 4092, 17), ("f32", 1024, 64), ("f32", 260, 64), ("f32", 4608, 3),
           # whole chunks, rows long and few enough for blocks of 32 rows
           ("bf16", 4608, 20), ("f16", 8192, 11), ("bf16", 4096, 36)]


@pytest.mark.parametrize("dtype,H,M", GENERAL)
def test_general_path_widths(coral, dtype, H, M):
    sizes = [1, 5, 127, 128, 129, 300, 90, 64, 260]
    cfg = HeadConfig(f"gen{H}", dtype, H, sum(sizes), len(sizes), 4, (M,), 12, 900 + H + M, True)
    check_all(coral, cfg, sizes, (M,))


@pytest.mark.parametrize("dtype,G,g,M", [("bf16", 65, 3, 40), ("f16", 128, 8, 64), ("f32", 200, 17, 33), ("bf16", 300, 70, 20)])
def test_general_path_many_groups(coral, dtype, G, g, M):
    sizes = [3 + (7 * n) % 40 for n in range(G)]
    cfg = HeadConfig(f"gengroups{G}", dtype, 1024, sum(sizes), G, g, (M,), 9, 940 + G, True)
    check_all(coral, cfg, sizes, (M,), dense=False)


@pytest.mark.parametrize("M,k,n_next", [(1, 1, 1), (3, 5, 15), (16, 64, 64), (17, 64, 64), (64, 64, 63), (64, 16, 64), (64, 16, 65)])
def test_tree_level_selection_and_ranking(coral, M, k, n_next):
    """Up to 64 kept nodes are selected, more are ranked: the same rules, bit for bit."""
    import oracle
    rng = np.random.default_rng(960 + M + k + n_next)
    logp = -np.sort(rng.random((M, k)).astype(np.float32).round(2) * 3, axis=1)   # rounded: ties
    ids = rng.integers(0, 1000, (M, k)).astype(np.int32)
    ids[M // 2, k // 2:] = -1                                                       # empty slots
    parent = (-rng.random(M).round(1) * 2).astype(np.float32)
    want = oracle.tree_expand(parent, ids, logp, n_next)
    got = coral.coral_tree_expand(torch.from_numpy(parent).cuda(), torch.from_numpy(ids).cuda(),
                                  torch.from_numpy(logp).cuda(), n_next)
    for a, b in zip(want, got):
        assert np.array_equal(np.asarray(a), b.cpu().numpy())


# Infinite logits (a vocabulary masked with -inf weights, sums beyond fp32): +-inf like any other
# value, also where a running sum keeps its rounding error.  "general": the tile kernels' general
# form, "small": its blocks of 32 rows, with whole and partly filled chunks of columns.
INFINITE = [("general", "bf16", 520, 64), ("general", "f32", 1024, 64), ("general", "f16", 1000, 50),
            ("general", "bf16", 5112, 33), ("small", "bf16", 8192, 12), ("small", "f16", 4608, 16),
            ("staged", "f32", 4608, 3), ("single", "bf16", 4096, 4)]


@pytest.mark.parametrize("form,dtype,H,M", INFINITE)
def test_infinite_logits(coral, form, dtype, H, M):
    sizes = [40, 130, 70, 300, 33, 64, 260, 128]
    G, g, k, V = len(sizes), 3, 64, sum(sizes)
    cfg = HeadConfig(f"inf_{form}", dtype, H, V, G, g, (M,), k, 980 + H + M, True)
    head = ragged_head(cfg, sizes)
    hidden = make_hidden(cfg, M, M)
    inf = {"bf16": (0x7f80, 0xff80), "f16": (0x7c00, 0xfc00), "f32": (np.float32(np.inf), np.float32(-np.inf))}[dtype]
    rng = np.random.default_rng(cfg.seed + 1)
    # one infinite weight in every ninth row (the sign of the logit is then that of the weight times
    # the token's value), everywhere from the first to the last column
    at = rng.permutation(V)[:V // 9]
    col = rng.integers(0, H, at.size)
    col[0], col[1] = 0, H - 1
    for n, (r, c) in enumerate(zip(at, col)):
        head.lm_W[r, c] = inf[n % 2]
    dh = DeviceHead(coral, head)
    d_hidden = coral.device_tensor(hidden, dtype)
    z = (d_hidden.double().cpu() @ dh.lm_W.double().cpu().t()).numpy()
    assert not np.isnan(z).any() and np.isinf(z).sum() == M * at.size
    group = np.empty(V, np.int64)
    group[head.group_rows] = np.repeat(np.arange(G), sizes)

    def best(values, groups=None):                     # the k best candidates, equal values by lower id
        cand = np.arange(V) if groups is None else np.flatnonzero(np.isin(group, groups))
        order = cand[np.lexsort((cand, -values[cand]))[:k]]
        return order, values[order]

    def agree(what, values, ids, val, sel=None):
        for m in range(M):
            print(f"{form} {dtype} H={H} {what}, token {m} of {M}", flush=True)
            want_ids, want = best(values[m], None if sel is None else sel[m])
            assert np.array_equal(np.isposinf(want), np.isposinf(val[m]))
            assert np.array_equal(np.isneginf(want), np.isneginf(val[m]))
            fin = np.isfinite(want)
            assert np.array_equal(ids[m][~fin], want_ids[~fin])      # (infinite values tie exactly)
            # 5e-5: the bound on log-probabilities of the parity tests, for values of this size
            assert (np.abs(val[m][fin] - want[fin]) <= 5e-5).all()
            assert (np.abs(val[m][fin] - values[m][ids[m][fin]]) <= 5e-5).all()

    ids, val, sel = run_grouped(coral, dh, hidden, g, k)
    agree("logits", z, ids, val, sel)
    agree("dense", z, *run_dense(coral, dh, hidden, k))

    # Masked rows: of every group all but the first 20, so that -inf reaches the list's end, in the
    # groups' sums of exp as well (a +inf there leaves its group's log-probabilities undefined).
    hid = np.abs(hidden) if dtype == "f32" else hidden & np.uint16(0x7fff)
    for n in range(G):
        masked = head.group_rows[head.group_offsets[n] + 20:head.group_offsets[n + 1]]
        head.lm_W[masked, rng.integers(0, H, masked.size)] = inf[1]
    head.lm_W[at, col] = inf[1]                        # (no +inf is left)
    dh = DeviceHead(coral, head)
    d_hid = coral.device_tensor(hid, dtype).double().cpu()
    z = (d_hid @ dh.lm_W.double().cpu().t()).numpy()
    s = (d_hid @ dh.gate_W.double().cpu().t()).numpy() + head.gate_bias
    router = s - np.log(np.exp(s).sum(axis=1, keepdims=True))
    lse = np.stack([np.log(np.exp(z[:, group == n]).sum(axis=1)) for n in range(G)], axis=1)
    assert not np.isnan(z).any() and not np.isposinf(z).any() and np.isfinite(lse).all()
    ids, val, sel = run_grouped(coral, dh, hid, g, k)
    agree("masked logits", z, ids, val, sel)
    ids, val, sel = run_logprob(coral, dh, hid, g, k)
    agree("masked log-probabilities", z + (router - lse)[:, group], ids, val, sel)


@pytest.mark.parametrize("dtype,H,G,v,g,k,Ms", [("f32", 256, 16, 598, 9, 16, (33, 32, 7)), ("bf16", 1024, 60, 190, 8, 16, (48, 33, 32, 1)),
                                                ("bf16", 8192, 32, 190, 4, 10, (20, 8, 9, 1)), ("f16", 1000, 20, 190, 2, 33, (64, 5, 40, 8))])
def test_one_workspace_for_several_token_counts(coral, dtype, H, G, v, g, k, Ms):
    """A workspace for the most tokens serves fewer, in any order and every output mode: the same
    bits as with a workspace of the call's own."""
    sizes = [v - 31 if n % 2 else v + 31 for n in range(G)]
    cfg = HeadConfig(f"ws{H}", dtype, H, sum(sizes), G, g, Ms, k, 990 + H, True)
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    code = {"bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16, "f32": coral.CORAL_F32}[dtype]
    ws = coral.alloc_workspace(max(Ms), H, cfg.V, G, g, k, code)
    for M in Ms:
        h = coral.device_tensor(make_hidden(cfg, M, M), dtype)
        for call in (lambda w: coral.coral_lmhead_grouped(h, dh.gate_W, dh.bias, dh.lm_W, dh.gi, g, k, workspace=w),
                     lambda w: coral.coral_lmhead_grouped_logprob(h, dh.gate_W, dh.bias, dh.lm_W, dh.gi, g, k, workspace=w),
                     lambda w: coral.coral_lmhead_dense(h, dh.lm_W, k, workspace=w)):
            print(f"case {dtype} H={H} M={M}", flush=True)
            for a, b in zip(call(None), call(ws)):
                assert torch.equal(a, b)


def test_log_probabilities_of_many_tokens_over_a_vocabulary_beyond_the_ranking_kernel(coral):
    """More than 32 tokens in the single launch: two passes of hidden vectors, pieces in memory."""
    cfg = HeadConfig("lpbig", "bf16", 64, 700_000, 16, 2, (40,), 8, 995, True)
    assert coral.coral_lmhead_logprob_path(40, 64, 700_000, 16, 2, 8, coral.CORAL_BF16) == 1
    dh = DeviceHead(coral, ragged_head(cfg, [43_750] * 16))
    hidden = make_hidden(cfg, 40, 1)
    check_logprob(dh, hidden, 2, 8, run_logprob(coral, dh, hidden, 2, 8))


def test_general_path_few_tokens_per_group(coral):
    """Rows beyond 8 KB: hardly more than one token per group (staged kernels), then two (tile
    kernels); the dense head with two tokens and three."""
    cfg = HeadConfig("few", "bf16", 4104, 45_056, 32, 4, (12, 16), 10, 996, True)
    assert coral.coral_lmhead_path(False, 12, cfg.H, cfg.V, cfg.G, cfg.g, cfg.k, coral.CORAL_BF16) == 0
    dh = DeviceHead(coral, ragged_head(cfg, [1408 + (n % 2 * 2 - 1) * 17 * (n // 2) for n in range(32)]))
    for M in (12, 16):
        hidden = make_hidden(cfg, M, M)
        print(f"case {cfg.name} M={M}", flush=True)
        check_grouped(dh, hidden, cfg.g, cfg.k, run_grouped(coral, dh, hidden, cfg.g, cfg.k))
        check_logprob(dh, hidden, cfg.g, cfg.k, run_logprob(coral, dh, hidden, cfg.g, cfg.k))
    for M in (2, 3):
        hidden = make_hidden(cfg, M, M)
        check_dense(dh, hidden, cfg.k, run_dense(coral, dh, hidden, cfg.k))


@pytest.mark.parametrize("dtype,H,M", [("bf16", 4608, 40), ("f16", 5120, 64), ("f32", 2304, 33)])
def test_small_blocks_of_a_group_with_two_passes_of_tokens(coral, dtype, H, M):
    """Blocks of 32 rows are chosen by the tokens per group on average; here every token chooses the
    same group, so its blocks come round twice, 32 tokens each."""
    sizes = [100, 70, 95, 161, 64, 33, 120, 96, 130]
    cfg = HeadConfig(f"pass{H}", dtype, H, sum(sizes), len(sizes), 1, (M,), 12, 997 + H, True)
    head = ragged_head(cfg, sizes)
    head.gate_bias[3] += 100.0
    dh = DeviceHead(coral, head)
    hidden = make_hidden(cfg, M, M)
    out = run_grouped(coral, dh, hidden, 1, 12)
    assert (out[2] == 3).all()
    check_grouped(dh, hidden, 1, 12, out)
    check_logprob(dh, hidden, 1, 12, run_logprob(coral, dh, hidden, 1, 12))


def test_tile_kernels_instead_of_lists(coral):
    """Many tokens whose candidates the single launch could not collect, dense and grouped."""
    cfg = HeadConfig("lists_f32", "f32", 232, 104_160, 20, 7, (62,), 10, 999, True)
    assert coral.coral_lmhead_path(False, 62, 232, cfg.V, 20, 7, 10, coral.CORAL_F32) == 0
    dh = DeviceHead(coral, ragged_head(cfg, [5208 + (n % 2 * 2 - 1) * n // 2 * 10 for n in range(20)]))
    hidden = make_hidden(cfg, 62, 1)
    check_grouped(dh, hidden, 7, 10, run_grouped(coral, dh, hidden, 7, 10))
    cfg = HeadConfig("lists_bf16", "bf16", 512, 40_000, 4, 2, (64,), 10, 1001, True)
    assert coral.coral_lmhead_path(True, 64, 512, cfg.V, 0, 0, 10, coral.CORAL_BF16) == 2
    dh = DeviceHead(coral, ragged_head(cfg, [10_000] * 4))
    hidden = make_hidden(cfg, 64, 1)
    check_dense(dh, hidden, 10, run_dense(coral, dh, hidden, 10))


@pytest.mark.parametrize("dtype,H,G,Ms", [("bf16", 4616, 200, (1, 6)), ("f32", 2564, 150, (2, 9)), ("f16", 8192, 100, (1, 9)),
                                          ("bf16", 5120, 48, (3, 6)), ("f32", 4096, 70, (1, 4))])
def test_rows_beyond_8_kb_with_many_groups(coral, dtype, H, G, Ms):
    """Both sides of the rule that keeps such rows in the single launch: groups and tokens."""
    sizes = [9 + (11 * n) % 50 for n in range(G)]
    cfg = HeadConfig(f"longgroups{H}", dtype, H, sum(sizes), G, 2, Ms, 8, 1003 + H, True)
    check_all(coral, cfg, sizes, Ms, dense=False)


@pytest.mark.parametrize("k", [10, 11, 33, 64])
@pytest.mark.parametrize("rows", [200, 3000, 9000, 17000])
def test_ranking_kernel_samples(coral, rows, k):
    """The ranking behind the tile kernels: 4 to 270 blocks per token (dense: up to 535) and every form
    of the bound; then equal logits, which no bound by value divides."""
    sizes = [rows + 61 * (n - 1) for n in range(4)]
    cfg = HeadConfig(f"rank{rows}", "bf16", 512, sum(sizes), 4, 2, (33,), k, 1010 + rows + k, True)
    assert coral.coral_lmhead_logprob_path(33, 512, cfg.V, 4, 2, k, coral.CORAL_BF16) == 2
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    hidden = make_hidden(cfg, 33, 1)
    check_grouped(dh, hidden, 2, k, run_grouped(coral, dh, hidden, 2, k))
    check_logprob(dh, hidden, 2, k, run_logprob(coral, dh, hidden, 2, k))
    check_dense(dh, hidden, k, run_dense(coral, dh, hidden, k))
    hidden = np.zeros((33, 512), np.uint16)
    check_dense(dh, hidden, k, run_dense(coral, dh, hidden, k))
    check_logprob(dh, hidden, 2, k, run_logprob(coral, dh, hidden, 2, k))


@pytest.mark.parametrize("dtype,H,M", [("bf16", 512, 34), ("f16", 1024, 40), ("bf16", 1536, 33), ("bf16", 2048, 64), ("f16", 2560, 48),
                                       ("bf16", 3072, 40)])
def test_blocks_in_halves(coral, dtype, H, M):
    """The tile path's last round of blocks in halves of 64 rows: one chunk of columns (never halved)
    to six, groups that end in either half, one of them with too many tokens; then all of one round and
    a rest in halves, grouped and dense."""
    sizes = [64, 65, 1, 127, 128, 129, 300, 192, 193, 90, 410, 260]
    cfg = HeadConfig(f"half{H}", dtype, H, sum(sizes), len(sizes), 2, (M,), 12, 1100 + H, True)
    head = ragged_head(cfg, sizes)
    head.gate_bias[6] += 2.0
    dh = DeviceHead(coral, head)
    hidden = make_hidden(cfg, M, M)
    assert coral.coral_lmhead_logprob_path(M, H, cfg.V, cfg.G, 2, 12, coral.CORAL_BF16) == 2
    check_grouped(dh, hidden, 2, 12, run_grouped(coral, dh, hidden, 2, 12))
    out = run_logprob(coral, dh, hidden, 2, 12)
    check_logprob(dh, hidden, 2, 12, out)
    assert all(np.array_equal(x, y) for x, y in zip(out, run_logprob(coral, dh, hidden, 2, 12)))


def test_a_whole_round_of_blocks_and_a_rest_in_halves(coral):
    cfg = HeadConfig("rest", "bf16", 1024, 40_100, 16, 4, (40,), 10, 1200, True)
    sizes = [2500] * 15 + [2600]
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    for M in (40, 32):
        hidden = make_hidden(cfg, M, M)
        check_logprob(dh, hidden, 4, 10, run_logprob(coral, dh, hidden, 4, 10))
        check_dense(dh, hidden, 10, run_dense(coral, dh, hidden, 10))


@pytest.mark.parametrize("M", [8, 9, 16, 17, 24, 25, 32])
def test_log_probabilities_where_many_tokens_share_a_group(coral, M):
    """The single launch's end in log-probability mode: two waves per (token, group) up to eight tokens
    of a group, one beyond, sixteen at a time."""
    sizes = [700, 90, 333, 64, 210, 8]
    cfg = HeadConfig(f"share{M}", "bf16", 512, sum(sizes), len(sizes), 2, (M,), 20, 1300 + M, True)
    head = ragged_head(cfg, sizes)
    head.gate_bias[2] += 100.0                         # in every token's selection
    dh = DeviceHead(coral, head)
    assert coral.coral_lmhead_logprob_path(M, 512, cfg.V, cfg.G, 2, 20, coral.CORAL_BF16) == 1
    hidden = make_hidden(cfg, M, M)
    out = run_logprob(coral, dh, hidden, 2, 20)
    assert (out[2] == 2).any(axis=1).all()
    check_logprob(dh, hidden, 2, 20, out)
    assert all(np.array_equal(x, y) for x, y in zip(out, run_logprob(coral, dh, hidden, 2, 20)))


@pytest.mark.parametrize("k", [1, 15, 16, 17, 31, 32, 33, 64])
@pytest.mark.parametrize("M", [1, 4, 5])
def test_few_batches_and_lists_fetched_in_one_trip(coral, M, k):
    """A small head: workgroups without a batch leave early, and the lists of the others are merged in
    one trip up to 512 entries."""
    cfg = HeadConfig(f"trip{k}", "f32", 256, 3510, 7, 1, (M,), k, 1400 + M + k, True)
    sizes = [495 + 2 * n for n in range(7)]
    sizes[-1] += 3510 - sum(sizes)
    check_all(coral, cfg, sizes, (M,))


@pytest.mark.parametrize("dtype,H,M", [("bf16", 8, 1), ("f16", 136, 2), ("bf16", 264, 15), ("f16", 1000, 16), ("bf16", 2568, 17), ("f16", 1160, 33),
                                       ("bf16", 1032, 49), ("f16", 520, 65), ("bf16", 5120, 3), ("bf16", 6016, 1), ("f16", 6016, 2),
                                       ("bf16", 7680, 1), ("f16", 8192, 3), ("bf16", 8192, 4), ("bf16", 3072, 8), ("bf16", 3584, 8), ("f16", 3584, 9),
                                       ("f32", 4, 1), ("f32", 1532, 5), ("f32", 1536, 4), ("f32", 1540, 5), ("f32", 1796, 32),
                                       ("f32", 1544, 40), ("f32", 1536, 64), ("f32", 1620, 130)])
def test_premix_of_any_width(coral, dtype, H, M):
    """The kernel for any width: the last 256-byte block and the last 16 features partly filled, fewer
    blocks than waves, one to four token tiles and several times 64 tokens, either side of its rule."""
    from coral_inputs import make_router_W1
    from oracle import compare
    cfg = HeadConfig(f"premix_any_{dtype}_{H}", dtype, H, 64, 2, 1, (M,), 4, 1500 + M, True)
    W1, hidden = make_router_W1(cfg), make_hidden(cfg, M, 0)
    print(f"case premix {dtype} H={H} M={M}", flush=True)
    u = coral.coral_router_premix(coral.device_tensor(hidden, dtype), coral.device_tensor(W1, dtype), "silu")
    raw = u.cpu().numpy() if dtype == "f32" else u.view(torch.int16).cpu().numpy().view(np.uint16)
    assert compare.check_premix(hidden, W1, dtype, "silu", raw).tokens == M


@pytest.mark.parametrize("dtype,H,V,M,k", [("bf16", 512, 8192, 16, 10), ("f16", 1000, 8300, 17, 1), ("bf16", 264, 9001, 33, 20), ("f32", 512, 8193, 24, 10),
                                           ("bf16", 1024, 8200, 15, 10), ("bf16", 512, 8191, 40, 10), ("f32", 516, 8250, 23, 4),
                                           ("f16", 1000, 9000, 24, 1), ("f32", 512, 9000, 24, 1), ("f32", 328, 8202, 32, 20)])
def test_dense_heads_with_many_tokens(coral, dtype, H, V, M, k):
    """Dense heads on either side of the line between the single launch and the tile kernels."""
    cfg = HeadConfig(f"dense{H}", dtype, H, V, 2, 1, (M,), k, 1600 + M, True)
    dh = DeviceHead(coral, ragged_head(cfg, [V // 2, V - V // 2]))
    hidden = make_hidden(cfg, M, M)
    check_dense(dh, hidden, k, run_dense(coral, dh, hidden, k))


@pytest.mark.parametrize("H,M", [(4096, 8), (4104, 16), (7168, 2), (8192, 64), (10248, 16)])
def test_premix_sums_on_the_matrix_cores(coral, H, M):
    """Values of u that rounding takes to the other of two 16-bit neighbours: their share is the mean
    error of the sums over the spacing of the results.  Sums of 128 to 160 products each, gathered in
    fp32, leave 6e-5 to 7.6e-5 of them here, as the vector units' do; one running sum per wave and
    feature leaves 8.8e-5 to 1.6e-4."""
    g = torch.Generator(device="cuda").manual_seed(5)
    wrong = total = 0
    for seed in range(2):
        W1 = (torch.randn(H, H, generator=g, device="cuda") * 0.02).bfloat16()
        hidden = torch.randn(1024, H, generator=g, device="cuda").bfloat16()
        u = torch.empty_like(hidden)
        print(f"case premix sums H={H} M={M} seed {seed}", flush=True)
        for m in range(0, 1024, M):
            coral.coral_router_premix(hidden[m:m + M], W1, "silu", out=u[m:m + M])
        y = torch.cat([hidden.double() @ W1[lo:lo + 1024].double().t() for lo in range(0, H, 1024)], dim=1)
        want = y / (1.0 + torch.exp(-y)) + hidden.double()
        wrong += int((u != want.bfloat16()).sum())
        total += u.numel()
    print(f"  {wrong} of {total}: {wrong / total:.2e}")
    assert wrong < 8e-5 * total


@pytest.mark.parametrize("dtype,H,V,M,path", [("bf16", 4096, 20000, 40, 2), ("f16", 4160, 20000, 24, 0), ("f32", 1536, 24000, 24, 0)])
def test_tile_kernels_past_the_caches_and_through_them(coral, dtype, H, V, M, path):
    """The tile kernels choose their loads by the rows that the tokens activate: more than 128 MB of all
    groups, then less of the two that a strong bias leaves."""
    cfg = HeadConfig(f"loads{H}", dtype, H, V, 8, 2, (M,), 10, 1700 + H, True)
    head = ragged_head(cfg, [V // 8] * 8)
    dt = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    assert coral.coral_lmhead_path(False, M, H, V, 8, 2, 10, dt) == path
    hidden = make_hidden(cfg, M, M)
    for strong in (0.0, 100.0):
        head.gate_bias[2:4] += strong
        dh = DeviceHead(coral, head)
        out = run_grouped(coral, dh, hidden, 2, 10)
        check_grouped(dh, hidden, 2, 10, out)
        row_bytes = H * (4 if dtype == "f32" else 2)
        activated = np.unique(out[2]).size * (V // 8) * row_bytes
        assert (activated < 128e6) == (strong > 0)


# H, groups, tokens where the single launch's gate is shared between the workgroups: both sides of a workgroup
# per group (256) and of the scores' words (4096), one (group, token) pair per workgroup to four per wave,
# rows of one to sixteen wave loads; the last two tokens counts of a line: shared and own on one workspace
SHARED_GATE = [("bf16", 8192, 8, (4, 1)), ("f16", 4096, 65, (1, 5, 16)), ("bf16", 4096, 300, (1, 3, 13, 14)),
               ("f32", 4096, 17, (5, 1)), ("f32", 1000, 64, (16, 20, 2)), ("bf16", 520, 128, (4, 32, 33)), ("f16", 6664, 40, (4, 2))]


@pytest.mark.parametrize("dtype,H,G,Ms", SHARED_GATE)
def test_gate_shared_between_workgroups(coral, dtype, H, G, Ms):
    sizes = [9 + (7 * n) % 11 for n in range(G)]
    V, g, k = sum(sizes), 3, 6
    cfg = HeadConfig(f"gate{G}", dtype, H, V, G, g, (1,), k, 900 + G, True)
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    code = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    ws = coral.alloc_workspace(max(Ms), H, V, G, g, k, code)
    for M in Ms + Ms:
        hidden = make_hidden(cfg, M, M)
        print(f"case {cfg.name} {dtype} H={H} M={M}", flush=True)
        assert coral.coral_lmhead_path(False, M, H, V, G, g, k, code) == 1
        d_hidden = coral.device_tensor(hidden, dtype)
        for logprob, check in ((False, check_grouped), (True, check_logprob)):
            out = coral.coral_lmhead_grouped(d_hidden, dh.gate_W, dh.bias, dh.lm_W, dh.gi, g, k, workspace=ws, logprob=logprob)
            torch.cuda.synchronize()
            check(dh, hidden, g, k, tuple(x.cpu().numpy() for x in out))


def test_shared_gate_with_scores_of_zero(coral):
    """All-zero hidden vectors: every score is +0, the word that stands for none; the lower groups win."""
    sizes = [40] * 48
    cfg = HeadConfig("gate0", "bf16", 8192, sum(sizes), 48, 4, (1,), 5, 930, True)
    head = ragged_head(cfg, sizes)
    head.gate_bias[:] = 0.0
    dh = DeviceHead(coral, head)
    for _ in range(2):
        ids, logits, sel = run_grouped(coral, dh, np.zeros((6, 8192), np.uint16), 4, 5)
        assert np.array_equal(sel, np.tile(np.arange(4), (6, 1))) and not logits.any()
        assert np.array_equal(ids, np.tile(np.sort(head.group_rows[:160])[:5], (6, 1)))


@pytest.mark.parametrize("dtype,H", [("bf16", 4224), ("f16", 4600), ("bf16", 4608), ("f32", 2112), ("f32", 2304)])
def test_rows_of_nine_segments(coral, dtype, H):
    """From a quarter of the ninth segment on, up to a whole one; the dense head up to seven tokens,
    log-probabilities up to eight."""
    sizes = [1, 2, 3, 15, 16, 17, 64, 130] + [40] * 25
    cfg = HeadConfig(f"nine{H}", dtype, H, sum(sizes), len(sizes), 4, (1,), 9, 950 + H, True)
    code = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    for M in (1, 3, 7, 8, 9):
        assert coral.coral_lmhead_path(False, M, H, cfg.V, cfg.G, 4, 9, code) == 1
        assert (coral.coral_lmhead_path(True, M, H, cfg.V, 0, 0, 9, code) == 1) == (M <= 7)
        assert (coral.coral_lmhead_logprob_path(M, H, cfg.V, cfg.G, 4, 9, code) == 1) == (M <= 8)
    check_all(coral, cfg, sizes, (1, 3, 7, 8, 9))


@pytest.mark.parametrize("dtype,H,M,path", [("bf16", 512, 37, 2), ("f16", 264, 64, 0), ("bf16", 1000, 38, 0), ("bf16", 512, 36, 1), ("f32", 512, 40, 1)])
def test_grouped_heads_with_many_tokens(coral, dtype, H, M, path):
    """Either side of the rule by tokens and storage type; whole and partly filled chunks."""
    sizes = [300 + 37 * n for n in range(20)]
    cfg = HeadConfig(f"many{H}", dtype, H, sum(sizes), 20, 3, (M,), 8, 980 + H + M, True)
    code = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    assert coral.coral_lmhead_path(False, M, H, cfg.V, 20, 3, 8, code) == path
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    hidden = make_hidden(cfg, M, M)
    check_grouped(dh, hidden, 3, 8, run_grouped(coral, dh, hidden, 3, 8))


# storage, H, groups, tokens: scores that are and are not a whole number of 16-byte words, more groups
# than workgroups, more than a wave's 256 words
GATE_ALONE = [("bf16", 8192, 40, 4), ("f16", 4096, 65, 5), ("bf16", 4096, 300, 13), ("f32", 1000, 64, 16), ("f16", 6664, 37, 3)]


@pytest.mark.parametrize("dtype,H,G,M", GATE_ALONE)
def test_shared_gate_where_workgroups_give_up(coral, dtype, H, G, M):
    """A workspace of which only the 512 bytes of control words were prepared: every workgroup computes
    the gate alone, with the bits of the shared one, and leaves the score words fit for sharing.  One
    request for the scores: who finds them all goes on, the others compute what is missing.  Undisturbed,
    the workgroups do not give up."""
    sizes = [9 + (7 * n) % 11 for n in range(G)]
    V, g, k = sum(sizes), 3, 6
    cfg = HeadConfig(f"alone{G}", dtype, H, V, G, g, (M,), k, 970 + G, True)
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    code = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    hidden = make_hidden(cfg, M, M)
    d_hidden = coral.device_tensor(hidden, dtype)
    routed = coral.device_tensor(make_hidden(cfg, M, M + 1), dtype)
    ws = coral.alloc_workspace(M, H, V, G, g, k, code)
    words = ws[:4 * (128 + 4096)].view(torch.int32)
    gave_up, polls = 2, 32
    workgroups = min(256, torch.cuda.get_device_properties(0).multi_processor_count)
    print(f"case {cfg.name} {dtype} H={H} M={M}", flush=True)

    def call(logprob, gate_hidden):
        out = coral.coral_lmhead_grouped(d_hidden, dh.gate_W, dh.bias, dh.lm_W, dh.gi, g, k, workspace=ws, logprob=logprob,
                                         gate_hidden=gate_hidden)
        return [x.cpu().numpy() for x in out]

    for logprob in (False, True):
        for gate_hidden in (None, routed):
            coral.coral_lmhead_workspace_init(ws)
            most = int(words[polls])
            for _ in range(4):
                shared = call(logprob, gate_hidden)
            assert int(words[gave_up]) < workgroups
            if gate_hidden is None:
                (check_logprob if logprob else check_grouped)(dh, hidden, g, k, tuple(shared))
            ws.fill_(0xAB)
            coral.coral_lmhead_workspace_init(ws[:512])
            assert int(words[polls]) == 0
            alone = call(logprob, gate_hidden)
            assert int(words[gave_up]) == workgroups and int(words[polls]) == most > 0
            assert not words[128:].any() and int(words[0]) == 0 and int(words[1]) == 0
            words[polls] = 1
            some = call(logprob, gate_hidden)
            words[polls] = most
            for out in (alone, some, call(logprob, gate_hidden)):
                assert all(np.array_equal(x, y) for x, y in zip(shared, out))
            assert not words[128:].any() and int(words[0]) == 0 and int(words[1]) == 0


def gate_is_shared(coral, dtype, H, G, M, k=2, g=2):
    """Whether the single launch shares the gate at these sizes: such a call is what marks the score words of
    a workspace as cleared (control word 32) whose first 512 bytes only were prepared."""
    code = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    sizes = [3] * G
    assert coral.coral_lmhead_path(False, M, H, sum(sizes), G, g, k, code) == 1
    dh = DeviceHead(coral, ragged_head(HeadConfig("which", dtype, H, sum(sizes), G, g, (M,), k, 5, True), sizes))
    ws = coral.alloc_workspace(M, H, sum(sizes), G, g, k, code)
    coral.coral_lmhead_workspace_init(ws[:512])
    hidden = coral.device_tensor(make_hidden(dh.head.cfg, M, M), dtype)
    coral.coral_lmhead_grouped(hidden, dh.gate_W, dh.bias, dh.lm_W, dh.gi, g, k, workspace=ws)
    return int(ws[:512].view(torch.int32)[32]) != 0


# either side of the bytes of a gate that up to three tokens share, and of the estimate that more go by
WHICH_GATE = [("bf16", 2776, 66, 1, False), ("bf16", 8192, 32, 1, True), ("bf16", 8192, 31, 1, False), ("f16", 2048, 70, 2, False),
              ("f16", 2048, 80, 2, True), ("bf16", 4096, 24, 3, False), ("bf16", 4096, 26, 3, True), ("f32", 2004, 52, 1, False),
              ("f32", 2048, 64, 1, True), ("bf16", 2048, 32, 8, False), ("bf16", 4096, 32, 8, True), ("bf16", 8192, 900, 5, False)]


@pytest.mark.parametrize("dtype,H,G,M,shared", WHICH_GATE)
def test_which_gates_are_shared(coral, dtype, H, G, M, shared):
    assert gate_is_shared(coral, dtype, H, G, M) == shared


# storage, H, groups, tokens, route with log-probabilities where every workgroup computes the gate on the matrix cores for itself: gates too
# small to be shared, and more scores than there are words for (rows of one, two and four passes of loads)
OWN_GATE = [("bf16", 2048, 32, 4, 1), ("f16", 2048, 32, 8, 1), ("bf16", 2048, 32, 16, 1), ("f16", 520, 64, 33, 0),
            ("bf16", 512, 1024, 5, 1), ("bf16", 4096, 300, 14, 1), ("f16", 3080, 830, 5, 1), ("bf16", 8192, 900, 5, 0)]


@pytest.mark.parametrize("dtype,H,G,M,logprob_path", OWN_GATE)
def test_own_gate_on_the_matrix_cores(coral, dtype, H, G, M, logprob_path):
    """Plain and routed, both output modes; that the gate was not shared is read from the workspace."""
    sizes = [20 + (7 * n) % 11 for n in range(G)]
    V, g, k = sum(sizes), 3, 6
    cfg = HeadConfig(f"own{G}", dtype, H, V, G, g, (M,), k, 990 + G + M, True)
    dh = DeviceHead(coral, ragged_head(cfg, sizes))
    h = dh.head
    code = {"bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    assert coral.coral_lmhead_path(False, M, H, V, G, g, k, code) == 1
    assert coral.coral_lmhead_logprob_path(M, H, V, G, g, k, code) == logprob_path
    hidden, gate_hidden = make_hidden(cfg, M, M), make_hidden(cfg, M, M + 1)
    d_hidden, d_gate_hidden = coral.device_tensor(hidden, dtype), coral.device_tensor(gate_hidden, dtype)
    ws = coral.alloc_workspace(M, H, V, G, g, k, code)
    ws.fill_(0xAB)
    coral.coral_lmhead_workspace_init(ws[:512])
    for logprob in (False, True):
        for seen, d_seen in ((hidden, None), (gate_hidden, d_gate_hidden)):
            print(f"case {cfg.name} {dtype} H={H} M={M} logprob={logprob} routed={d_seen is not None}", flush=True)
            out = coral.coral_lmhead_grouped(d_hidden, dh.gate_W, dh.bias, dh.lm_W, dh.gi, g, k, workspace=ws, logprob=logprob,
                                             gate_hidden=d_seen)
            out = [x.cpu().numpy() for x in out]
            check = compare.check_grouped_logprob if logprob else compare.check_grouped
            rep = check(hidden, h.gate_W, h.gate_bias, h.lm_W, h.group_offsets, h.group_rows, g, k, dtype, *out,
                        gate_hidden=None if d_seen is None else seen)
            assert rep.max_abs_err <= (TIGHT_LOGP_ERR if logprob else TIGHT_LOGIT_ERR)[dtype]
            assert int(ws[:512].view(torch.int32)[32]) == 0        # no call that shares the gate
