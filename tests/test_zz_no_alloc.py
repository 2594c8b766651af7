"""The entry point that allocates nothing (coral_lmhead_grouped_noalloc) against
coral_lmhead_grouped, through the C ABI on a real MI355X: same kernels on the library's
static scratch array instead of a caller's workspace, so ids, logits and groups must agree
bit for bit.  Every case makes two calls in a row, the second with a smaller input: the
array keeps what the first call left there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from coral_inputs import CONFIGS, HeadConfig, make_head, make_hidden  # noqa: E402


@pytest.fixture(scope="module")
def coral():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_16880_amd as c
    return c


def upload(coral, head):
    c = head.cfg
    return (coral.device_tensor(head.gate_W, c.dtype), coral.device_tensor(head.lm_W, c.dtype),
            None if head.gate_bias is None else torch.from_numpy(head.gate_bias).cuda(),
            coral.GroupIndex(head.group_offsets, head.group_rows))


def both(coral, cfg, dev, M, g, k, batch):
    """(reference entry point's outputs, new entry point's outputs) for one seeded batch."""
    gate_W, lm_W, bias, gi = dev
    d_hidden = coral.device_tensor(make_hidden(cfg, M, batch), cfg.dtype)
    want = coral.coral_lmhead_grouped(d_hidden, gate_W, bias, lm_W, gi, g, k)
    ids = torch.full((M, k), -5, dtype=torch.int32, device="cuda")
    z = torch.full((M, k), float("nan"), device="cuda")
    sel = torch.full((M, g), -5, dtype=torch.int32, device="cuda")
    coral.coral_lmhead_grouped_noalloc(d_hidden, gate_W, bias, lm_W, gi, g, k, ids, z, sel)
    torch.cuda.synchronize()
    return want, (ids, z, sel)


CASES = [
    # (config, expected path, (M, g, k) of the first call, of the second, smaller one)
    (CONFIGS["llama3_8b"].scaled(V=32 * 203), 1, (8, 4, 10), (3, 2, 7)),
    (CONFIGS["tiny_f32"], 1, (4, 2, 8), (1, 1, 3)),
    (CONFIGS["wide_tree"].scaled(V=64 * 126), 2, (64, 8, 16), (40, 8, 16)),
    (CONFIGS["llama3_8b"].scaled(name="llama3_f16_h4160", dtype="f16", V=32 * 203, H=4160), 0,
     (8, 4, 10), (2, 4, 10)),
]


@pytest.mark.parametrize("cfg,path,first,second", CASES,
                         ids=lambda x: x.name if isinstance(x, HeadConfig) else None)
def test_noalloc_matches_grouped_on_two_calls_in_a_row(coral, cfg, path, first, second):
    dt = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[cfg.dtype]
    dev = upload(coral, make_head(cfg))
    for call, (M, g, k) in enumerate((first, second)):
        if call == 0:
            assert coral.coral_lmhead_path(False, M, cfg.H, cfg.V, cfg.G, g, k, dt) == path
        print(f"case {cfg.name} call {call}: M={M} g={g} k={k}", flush=True)
        want, got = both(coral, cfg, dev, M, g, k, batch=call)
        for name, a, b in zip(("ids", "logits", "groups"), want, got):
            assert torch.equal(a, b), f"{name} differ on call {call}"


def test_noalloc_at_full_size_then_a_smaller_vocabulary(coral):
    """The headline shape with 16 tokens (7 MB of scratch), then one token, then another,
    smaller head: a different layout over the same array."""
    cfg = CONFIGS["llama3_8b"]
    dev = upload(coral, make_head(cfg))
    for call, M in enumerate((16, 1)):
        print(f"case {cfg.name} M={M}", flush=True)
        want, got = both(coral, cfg, dev, M, cfg.g, cfg.k, batch=call)
        for a, b in zip(want, got):
            assert torch.equal(a, b)
    del dev
    torch.cuda.empty_cache()
    small = CONFIGS["llama2_7b"].scaled(V=16 * 250)
    want, got = both(coral, small, upload(coral, make_head(small)), 4, small.g, small.k, batch=0)
    for a, b in zip(want, got):
        assert torch.equal(a, b)


def test_noalloc_with_own_and_shared_gate_in_turn(coral):
    """The scores' words are prepared only by calls that use them, whatever lay there before."""
    tree, llama = CONFIGS["wide_tree"].scaled(V=64 * 126), CONFIGS["llama3_8b"].scaled(V=32 * 203)
    heads = {c.name: upload(coral, make_head(c)) for c in (tree, llama)}
    for call, (cfg, M) in enumerate(((tree, 64), (llama, 8), (llama, 1), (llama, 16), (tree, 40), (llama, 2), (llama, 5))):
        print(f"case {cfg.name} M={M}", flush=True)
        want, got = both(coral, cfg, heads[cfg.name], M, cfg.g, cfg.k, batch=call)
        for a, b in zip(want, got):
            assert torch.equal(a, b)


def test_noalloc_refuses_shapes_beyond_its_scratch(coral):
    """64 tokens x 16 candidates at the full vocabulary need 37 MB: refused before any launch
    (the weights here are a small dummy; the size check sees the declared shape only)."""
    cfg = CONFIGS["wide_tree"]
    need = coral.coral_lmhead_workspace_bytes(64, cfg.H, cfg.V, cfg.G, cfg.g, cfg.k, coral.CORAL_BF16)
    assert need > coral.NOALLOC_SCRATCH_BYTES
    head = make_head(cfg.scaled(V=64 * 126))
    gate_W, _, bias, _ = upload(coral, head)
    rows = np.arange(cfg.V, dtype=np.int32)
    offsets = (np.arange(cfg.G + 1) * cfg.v).astype(np.int32)
    gi = coral.GroupIndex(offsets, rows, validate=False)
    # a [V,H] weight tensor of 1 GB just to be refused would be wasteful: the C ABI is called
    # directly with a small buffer's address, which the refused call never reads
    lm_W = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    d_hidden = coral.device_tensor(make_hidden(cfg, 64, 0), cfg.dtype)
    ids = torch.empty((64, cfg.k), dtype=torch.int32, device="cuda")
    z = torch.empty((64, cfg.k), device="cuda")
    st = coral._L.coral_lmhead_grouped_noalloc(
        d_hidden.data_ptr(), gate_W.data_ptr(), bias.data_ptr(), lm_W.data_ptr(), gi.struct(),
        64, cfg.H, cfg.V, cfg.g, cfg.k, coral.CORAL_BF16, ids.data_ptr(), z.data_ptr(), None, None)
    assert st == 5                                       # CORAL_ERR_WORKSPACE
    torch.cuda.synchronize()


def test_noalloc_under_graph_capture(coral):
    """The callers it is for: captured after one eager call (which looks the array up),
    replayed with eager work in between, every replay equal to the eager result."""
    cfg = CONFIGS["llama3_8b"].scaled(V=32 * 501)
    gate_W, lm_W, bias, gi = upload(coral, make_head(cfg))
    M = 4
    d_hidden = coral.device_tensor(make_hidden(cfg, M, 1), cfg.dtype)
    want = coral.coral_lmhead_grouped(d_hidden, gate_W, bias, lm_W, gi, cfg.g, cfg.k)
    ids = torch.empty((M, cfg.k), dtype=torch.int32, device="cuda")
    z = torch.empty((M, cfg.k), device="cuda")
    sel = torch.empty((M, cfg.g), dtype=torch.int32, device="cuda")

    def call():
        coral.coral_lmhead_grouped_noalloc(d_hidden, gate_W, bias, lm_W, gi, cfg.g, cfg.k, ids, z, sel)

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
        call()
    for rep in range(3):
        ids.fill_(-1), z.zero_(), sel.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(want, (ids, z, sel)):
            assert torch.equal(a, b), rep


# The general path's tile kernels (more than eight tokens): their arrays fit the scratch; or they do
# not, while the staged lists by which the shape is accepted do, and the tokens go in batches.
GENERAL = [("bf16", 1664, 6400, 16, 2, 10, 40), ("f16", 1000, 16000, 32, 3, 4, 64), ("f32", 2056, 4096, 16, 2, 8, 33),
           ("bf16", 1664, 50272, 16, 2, 10, 40), ("bf16", 2568, 100352, 64, 4, 2, 33), ("f32", 2308, 50272, 16, 2, 3, 64),
           ("f32", 232, 104160, 20, 7, 3, 62)]


@pytest.mark.parametrize("dtype,H,V,G,g,k,M", GENERAL)
def test_noalloc_on_the_general_paths_tile_kernels(coral, dtype, H, V, G, g, k, M):
    dt = {"f32": coral.CORAL_F32, "bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    cfg = HeadConfig(f"general{H}", dtype, H, V, G, g, (M,), k, 1000 + H, True, bias_std=0.5)
    assert coral.coral_lmhead_path(False, M, H, V, G, g, k, dt) == 0
    dev = upload(coral, make_head(cfg))
    for m in (M, M - 7):
        print(f"case {dtype} H={H} V={V} M={m}", flush=True)
        want, got = both(coral, cfg, dev, m, g, k, batch=m)
        for name, a, b in zip(("ids", "logits", "groups"), want, got):
            assert torch.equal(a, b), f"{name} differ with {m} tokens"


# The most tokens that the scratch takes: tile path with 128-row blocks, with 32-row blocks (whose
# statistics make the tokens go in batches), and a narrow head that the single-launch kernel runs.
LIMITS = [("bf16", 4096, 32000, 16, 2, 10, 60, 2), ("f16", 4096, 32000, 32, 4, 10, 56, 2),
          ("bf16", 4608, 56358, 93, 1, 4, 30, 2), ("bf16", 512, 32000, 16, 2, 64, 16, 1)]


@pytest.mark.parametrize("dtype,H,V,G,g,k,M,path", LIMITS)
def test_noalloc_at_the_limits_of_its_scratch(coral, dtype, H, V, G, g, k, M, path):
    code = {"bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    assert coral.coral_lmhead_path(False, M, H, V, G, g, k, code) == path
    print(f"case {dtype} H={H} V={V} M={M}", flush=True)
    torch.manual_seed(H + M)
    t = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    lm_W = (torch.randn(V, H, device="cuda", dtype=t)).mul_(0.02)
    gate_W = (torch.randn(G, H, device="cuda", dtype=t)).mul_(0.02)
    hidden = torch.randn(M, H, device="cuda", dtype=t)
    gi = coral.GroupIndex((np.arange(G + 1) * (V // G)).astype(np.int32), np.random.default_rng(1).permutation(V))
    want = coral.coral_lmhead_grouped(hidden, gate_W, None, lm_W, gi, g, k)
    ids = torch.full((M, k), -5, dtype=torch.int32, device="cuda")
    z = torch.full((M, k), float("nan"), device="cuda")
    sel = torch.full((M, g), -5, dtype=torch.int32, device="cuda")
    coral.coral_lmhead_grouped_noalloc(hidden, gate_W, None, lm_W, gi, g, k, ids, z, sel)
    torch.cuda.synchronize()
    for a, b in zip(want, (ids, z, sel)):
        assert torch.equal(a, b)


# Plain tile path, more tokens than the scratch takes at once (its logits), groups of uneven size and
# popularity: which blocks the last round holds differs from batch to batch.
BATCHED = [("bf16", 1024, 66000, 4, 2, 8, 48), ("f16", 1024, 100000, 8, 3, 4, 48), ("bf16", 1536, 100000, 4, 2, 8, 33)]


@pytest.mark.parametrize("dtype,H,V,G,g,k,M", BATCHED)
def test_noalloc_in_batches_on_the_tile_path(coral, dtype, H, V, G, g, k, M):
    code = {"bf16": coral.CORAL_BF16, "f16": coral.CORAL_F16}[dtype]
    assert coral.coral_lmhead_path(False, M, H, V, G, g, k, code) == 2
    assert M * V * 4 > coral.NOALLOC_SCRATCH_BYTES
    torch.manual_seed(H + M)
    t = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    lm_W = (torch.randn(V, H, device="cuda", dtype=t)).mul_(0.02)
    gate_W = (torch.randn(G, H, device="cuda", dtype=t)).mul_(0.02)
    bias = torch.zeros(G, device="cuda")
    bias[G - 1] = 1.5
    cuts = np.arange(G + 1) * (V // G)
    cuts[1:-1:2] += 200
    gi = coral.GroupIndex(cuts.astype(np.int32), np.random.default_rng(1).permutation(V).astype(np.int32))
    for call in range(3):
        print(f"case {dtype} H={H} V={V} M={M} call {call}", flush=True)
        hidden = torch.randn(M, H, device="cuda", dtype=t)
        want = coral.coral_lmhead_grouped(hidden, gate_W, bias, lm_W, gi, g, k)
        ids = torch.full((M, k), -5, dtype=torch.int32, device="cuda")
        z = torch.full((M, k), float("nan"), device="cuda")
        sel = torch.full((M, g), -5, dtype=torch.int32, device="cuda")
        coral.coral_lmhead_grouped_noalloc(hidden, gate_W, bias, lm_W, gi, g, k, ids, z, sel)
        torch.cuda.synchronize()
        for name, a, b in zip(("ids", "logits", "groups"), want, (ids, z, sel)):
            assert torch.equal(a, b), name
