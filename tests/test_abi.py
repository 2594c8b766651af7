"""Host-side checks of the C ABI (no GPU): the library loads, exports every symbol
the header declares, and rejects bad arguments before anything is enqueued."""
import ctypes
import os
import re

import numpy as np
import pytest
import torch

import paper_2502_16880_amd as coral

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "coral_lmhead.h")

OK, NULL, SHAPE, GROUP_INDEX, UNSUPPORTED, WORKSPACE, HIP = range(7)
F32, BF16, F16 = 0, 1, 2
FAKE = 0x7000_0000_1000          # never dereferenced: every check below fails before a launch


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(coral_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert {"coral_lmhead_grouped", "coral_lmhead_dense", "coral_lmhead_workspace_bytes",
            "coral_lmhead_workspace_init", "coral_lmhead_grouped_profiled",
            "coral_lmhead_dense_profiled",
            "coral_group_index_validate", "coral_status_string"} <= set(names)
    lib = ctypes.CDLL(coral.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), f"{n} declared in the header but not exported"


def test_probe_read_checks_its_arguments_on_the_host():
    L = coral._L
    assert L.coral_probe_read(None, 16384, 16, None, 1, 1) == 1               # CORAL_ERR_NULL
    assert L.coral_probe_read(4096, 16384, 16, None, None, 1) == 1
    assert L.coral_probe_read(4096, 1000, 16, None, 1, 1) == 2                # CORAL_ERR_SHAPE
    assert L.coral_probe_read(4096, 16384, 17, None, 1, 1) == 2
    assert L.coral_probe_read(4100, 16384, 16, None, 1, 1) == 4               # CORAL_ERR_UNSUPPORTED


def test_status_strings():
    seen = {coral.coral_status_string(i) for i in range(7)}
    assert len(seen) == 7 and coral.coral_status_string(0) == "ok"
    assert "unknown" in coral.coral_status_string(99)


def test_group_index_validate():
    L = coral._L
    off = np.array([0, 3, 6], dtype=np.int32)
    rows = np.array([5, 0, 2, 1, 4, 3], dtype=np.int32)
    v = lambda o, r, G, V: L.coral_group_index_validate(o.ctypes.data, r.ctypes.data, G, V)
    assert v(off, rows, 2, 6) == OK
    assert L.coral_group_index_validate(None, rows.ctypes.data, 2, 6) == NULL
    assert v(off, rows, 0, 6) == SHAPE
    bad = rows.copy(); bad[0] = 0
    assert v(off, bad, 2, 6) == GROUP_INDEX            # id 0 twice, id 5 missing
    bad = rows.copy(); bad[1] = 6
    assert v(off, bad, 2, 6) == GROUP_INDEX            # id out of range
    assert v(np.array([0, 4, 3], np.int32), rows, 2, 6) == GROUP_INDEX   # not ascending / end != V
    assert v(np.array([1, 3, 6], np.int32), rows, 2, 6) == GROUP_INDEX
    ragged = np.array([0, 1, 6], dtype=np.int32)       # ragged groups are a valid partition
    assert v(ragged, rows, 2, 6) == OK


def test_path_selection_covers_the_three_paths():
    path = coral.coral_lmhead_path
    assert path(False, 1, 4096, 128256, 32, 4, 10, BF16) == 1      # Llama3 shape, one token
    assert path(False, 16, 4096, 128256, 32, 4, 10, BF16) == 1
    assert path(False, 64, 4096, 128256, 64, 8, 16, BF16) == 2     # wide tree: hidden exceeds LDS
    assert path(True, 16, 4096, 128256, 0, 0, 10, BF16) == 2       # dense, many tokens
    assert path(True, 8, 4096, 32000, 0, 0, 10, BF16) == 1         # ... but a small vocabulary
    assert path(False, 64, 4160, 128256, 64, 8, 16, BF16) == 0     # H not a multiple of 512
    assert path(True, 1, 4096, 128256, 0, 0, 10, BF16) == 1
    assert path(False, 64, 512, 1040, 8, 1, 64, BF16) == 2         # k = 64 on the tile path too
    assert path(False, 4, 256, 8192, 16, 2, 8, F32) == 1
    assert path(True, 64, 4096, 8192, 0, 0, 8, F32) == 0           # fp32 rows longer than 8 KB
    assert path(True, 64, 8192, 8192, 0, 0, 8, F32) == -1          # ... than the staged path's LDS
    assert path(False, 65, 256, 8192, 16, 2, 8, F32) == -1


def test_logprob_path_selection():
    lp = coral.coral_lmhead_logprob_path
    assert lp(1, 4096, 128256, 32, 4, 10, BF16) == 1               # Llama3 shape
    assert lp(16, 4096, 128256, 32, 4, 10, BF16) == 1
    assert lp(16, 3584, 152064, 32, 4, 10, BF16) == 1              # Qwen shape
    assert lp(64, 4096, 128256, 64, 8, 16, BF16) == 2              # wide tree: hidden exceeds LDS
    assert lp(64, 4160, 128256, 64, 8, 16, BF16) == 0              # ... and H not a multiple of 512
    assert lp(64, 4096, 128256, 128, 8, 16, BF16) == 0             # tile path ranks 64 groups at most
    assert lp(20, 256, 8192, 128, 4, 8, F32) == 0                  # 80 groups may be active
    assert lp(2, 256, 8192, 64, 17, 8, F32) == 0                   # 17 lists per token
    assert lp(65, 256, 8192, 16, 2, 8, F32) == -1


def test_workspace_init_rejects_bad_arguments():
    L = coral._L
    assert L.coral_lmhead_workspace_init(None, 4096, None) == WORKSPACE
    assert L.coral_lmhead_workspace_init(FAKE + 8, 4096, None) == WORKSPACE
    assert L.coral_lmhead_workspace_init(FAKE, 16, None) == WORKSPACE


def test_workspace_bytes():
    wb = coral.coral_lmhead_workspace_bytes
    a = wb(1, 4096, 128256, 32, 4, 10, BF16)
    b = wb(16, 4096, 128256, 32, 4, 10, BF16)
    assert 0 < a < b
    assert wb(4, 256, 8192, 0, 0, 8, F32) > 0          # dense
    assert wb(0, 256, 8192, 16, 2, 8, F32) == 0
    assert wb(4, 256, 8192, 16, 0, 8, F32) == 0        # G without g
    assert wb(4, 256, 8192, 4, 5, 8, F32) == 0         # g > G
    assert b % 256 == 0
    # shapes that can take the matrix-core path carry its logits buffer, 512 B per (128-row
    # block, token) with V / 128 + G + 1 blocks; shapes that cannot (one token; fp32) do not
    z_wide = (128256 // 128 + 64 + 1) * 64 * 512
    assert wb(64, 4096, 128256, 64, 8, 16, BF16) - wb(64, 4096, 128256, 64, 8, 16, F32) >= z_wide
    # (the dense head takes that path from 8 tokens on: a workspace for 8 tokens serves it too)
    assert wb(8, 4096, 128256, 32, 4, 10, BF16) - wb(7, 4096, 128256, 32, 4, 10, BF16) >= (128256 // 128 + 32 + 1) * 8 * 512


class Call:
    """A grouped call with plausible arguments; tests override one at a time."""

    def __init__(self):
        self.G, self.v = 16, 512
        self.off = (np.arange(self.G + 1) * self.v).astype(np.int32)
        self.a = dict(hidden=FAKE, gate_W=FAKE + 0x100000, gate_bias=None, lm_W=FAKE + 0x200000,
                      M=4, H=256, V=8192, g=2, k=8, dt=F32, ids=FAKE + 0x300000,
                      logits=FAKE + 0x400000, sel=None, ws=FAKE + 0x500000, ws_bytes=1 << 30)
        self.gi = coral._GroupIndexStruct(self.G, self.off.ctypes.data, FAKE + 0x600000,
                                          FAKE + 0x700000)

    def grouped(self, gi="default", **kw):
        a = dict(self.a, **kw)
        gip = ctypes.byref(self.gi) if gi == "default" else gi
        return coral._L.coral_lmhead_grouped(a["hidden"], a["gate_W"], a["gate_bias"], a["lm_W"],
                                             gip, a["M"], a["H"], a["V"], a["g"], a["k"], a["dt"],
                                             a["ids"], a["logits"], a["sel"], a["ws"],
                                             a["ws_bytes"], None)

    def dense(self, **kw):
        a = dict(self.a, **kw)
        return coral._L.coral_lmhead_dense(a["hidden"], a["lm_W"], a["M"], a["H"], a["V"], a["k"],
                                           a["dt"], a["ids"], a["logits"], a["ws"], a["ws_bytes"],
                                           None)


@pytest.mark.parametrize("kw,want", [
    (dict(hidden=None), NULL), (dict(gate_W=None), NULL), (dict(lm_W=None), NULL),
    (dict(ids=None), NULL), (dict(logits=None), NULL),
    (dict(M=0), SHAPE), (dict(k=0), SHAPE), (dict(g=0), SHAPE), (dict(g=17), SHAPE),
    (dict(dt=7), SHAPE), (dict(V=8191), GROUP_INDEX),
    (dict(M=65), UNSUPPORTED), (dict(k=65), UNSUPPORTED),
    (dict(H=254), UNSUPPORTED), (dict(H=260, dt=BF16), UNSUPPORTED),
    (dict(hidden=FAKE + 8), UNSUPPORTED), (dict(lm_W=FAKE + 4), UNSUPPORTED),
    (dict(gate_W=FAKE + 2), UNSUPPORTED),
    (dict(ws=None), WORKSPACE), (dict(ws=FAKE + 64), WORKSPACE), (dict(ws_bytes=1024), WORKSPACE),
])
def test_grouped_rejects_bad_arguments_before_any_launch(kw, want):
    assert Call().grouped(**kw) == want


def test_grouped_group_index_errors():
    c = Call()
    assert c.grouped(gi=None) == NULL
    c.gi.group_rows = None
    assert c.grouped() == NULL
    c = Call()
    c.off[3] = c.off[2] - 1                            # descending offsets
    assert c.grouped() == GROUP_INDEX
    c = Call()
    c.gi.G = 2000
    assert c.grouped(g=2) in (UNSUPPORTED, SHAPE)
    c = Call()
    c.off[0] = 1
    assert c.grouped() == GROUP_INDEX


def test_k_larger_than_the_candidate_count():
    c = Call()
    c.off[:] = [0, 3, 6] + list(range(7, 7 + 13)) + [8192]    # two groups of 3 rows, many of 1
    assert c.grouped(g=2, k=3) == SHAPE                # the two smallest groups hold 2 rows
    assert c.grouped(g=2, k=2, ws=None) == WORKSPACE   # k = 2 passes that check


@pytest.mark.parametrize("kw,want", [
    (dict(hidden=None), NULL), (dict(lm_W=None), NULL), (dict(ids=None), NULL),
    (dict(M=0), SHAPE), (dict(k=0), SHAPE), (dict(V=4, k=8), SHAPE),
    (dict(M=65), UNSUPPORTED), (dict(k=65), UNSUPPORTED), (dict(H=258), UNSUPPORTED),
    (dict(ws=None), WORKSPACE), (dict(ws_bytes=16), WORKSPACE),
])
def test_dense_rejects_bad_arguments_before_any_launch(kw, want):
    assert Call().dense(**kw) == want


def test_binding_rejects_host_tensors_and_mixed_dtypes():
    import torch
    h = torch.zeros(2, 64)
    with pytest.raises(ValueError):
        coral.coral_lmhead_dense(h, torch.zeros(128, 64), 4,
                                 topk_ids=torch.zeros(2, 4, dtype=torch.int32),
                                 topk_logits=torch.zeros(2, 4),
                                 workspace=torch.zeros(1 << 20, dtype=torch.uint8))
    with pytest.raises(TypeError):
        coral.coral_lmhead_dense(h, torch.zeros(128, 64, dtype=torch.bfloat16), 4)
    with pytest.raises(TypeError):
        coral.coral_lmhead_dense(h.double(), torch.zeros(128, 64).double(), 4)


def test_rows_too_long_for_every_path_are_refused_before_any_launch():
    """A shape that only the staged path could take (H no multiple of 512) and whose batch of
    eight token vectors does not fit LDS: the path query says -1 and the call returns
    UNSUPPORTED with nothing enqueued (the fake pointers would fault otherwise)."""
    path, lp = coral.coral_lmhead_path, coral.coral_lmhead_logprob_path
    assert path(False, 8, 10248, 8192, 16, 2, 8, BF16) == -1
    assert path(True, 8, 10248, 8192, 0, 0, 8, BF16) == -1
    assert lp(8, 10248, 8192, 16, 2, 8, BF16) == -1
    assert path(False, 4, 10248, 8192, 16, 2, 8, BF16) == 0        # four token vectors do fit
    assert path(False, 8, 10240, 8192, 16, 2, 8, BF16) == 2        # whole 512-column chunks: tiles
    c = Call()
    assert c.grouped(M=8, H=10248, dt=BF16) == UNSUPPORTED
    assert c.dense(M=8, H=10248, dt=BF16) == UNSUPPORTED


def test_control_words_do_not_overlap(tmp_path):
    """The kernels' arrival counters and queues share the first words of the workspace; the
    map (csrc/control_words.h) is compiled here with the host compiler and checked: entries
    disjoint, inside the area that coral_lmhead_workspace_init zeroes, and the workspace of
    every shape at least that large."""
    import subprocess
    src = tmp_path / "ctrl.cpp"
    src.write_text('#include <cstdio>\n#include "control_words.h"\n'
                   'int main() { std::printf("words %d\\n", coral_ctrl::kWords);\n'
                   '  for (int i = 0; i < coral_ctrl::kMapEntries; ++i)\n'
                   '    std::printf("%s %d %d\\n", coral_ctrl::kMap[i].name, coral_ctrl::kMap[i].first_word,\n'
                   '                coral_ctrl::kMap[i].n_words);\n  return 0; }\n')
    exe = tmp_path / "ctrl"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2502_16880_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    words = int(lines[0].split()[1])
    entries = [(p[0], int(p[1]), int(p[2])) for p in (l.split() for l in lines[1:] if l.strip())]
    assert len(entries) >= 4 and len({e[0] for e in entries}) == len(entries)
    owner = {}
    for name, first, n in entries:
        assert n >= 1 and 0 <= first and first + n <= words, name
        for w in range(first, first + n):
            assert w not in owner, f"word {w}: {name} overlaps {owner.get(w)}"
            owner[w] = name
    names = {e[0]: e for e in entries}
    assert names["logprob_group_arrival"][2] >= 64          # one counter per activated group
    assert coral.coral_lmhead_workspace_bytes(1, 8, 1, 0, 0, 1, BF16) >= 4 * words
    # the preparation call insists on the whole area
    assert coral._L.coral_lmhead_workspace_init(FAKE, 4 * words - 4, None) == WORKSPACE


def test_noalloc_entry_point_checks_arguments_and_size_before_touching_the_device():
    """coral_lmhead_grouped_noalloc: the same argument errors as coral_lmhead_grouped, and a
    shape whose scratch need exceeds the library's static array is refused (WORKSPACE) with
    nothing looked up or enqueued."""
    c = Call()

    def noalloc(**kw):
        a = dict(c.a, **kw)
        return coral._L.coral_lmhead_grouped_noalloc(
            a["hidden"], a["gate_W"], a["gate_bias"], a["lm_W"], ctypes.byref(c.gi), a["M"], a["H"],
            a["V"], a["g"], a["k"], a["dt"], a["ids"], a["logits"], a["sel"], None)

    assert noalloc(hidden=None) == NULL
    assert noalloc(ids=None) == NULL
    assert noalloc(M=0) == SHAPE
    assert noalloc(M=65) == UNSUPPORTED
    assert noalloc(H=254) == UNSUPPORTED
    assert noalloc(g=17) == SHAPE
    # 64 tokens x 64 candidates: the published lists alone are 8 MiB
    assert coral.coral_lmhead_workspace_bytes(64, 256, 8192, 16, 2, 64, F32) > coral.NOALLOC_SCRATCH_BYTES
    assert noalloc(M=64, k=64) == WORKSPACE
    header = open(HEADER).read()
    m = re.search(r"#define\s+CORAL_NOALLOC_SCRATCH_BYTES\s+\((\d+)u\s*<<\s*(\d+)\)", header)
    assert m and int(m.group(1)) << int(m.group(2)) == coral.NOALLOC_SCRATCH_BYTES


def noalloc_status(M, H, V, G, g, k, dt):
    """Status of coral_lmhead_grouped_noalloc with made-up addresses.  Only without a GPU: a shape
    that passes the size check then stops where the scratch array's address is looked up."""
    off = (np.arange(G + 1, dtype=np.int64) * V // G).astype(np.int32)
    gi = coral._GroupIndexStruct(G, off.ctypes.data, FAKE + 0x600000, FAKE + 0x700000)
    return coral._L.coral_lmhead_grouped_noalloc(FAKE, FAKE + 0x100000, None, FAKE + 0x200000, ctypes.byref(gi), M, H,
                                                 V, g, k, dt, FAKE + 0x300000, FAKE + 0x400000, None, None)


# (H, V, G, g, k, storage) and the most tokens that the static scratch takes: counted by the tile
# path's arrays (whole 512-column chunks, rows beyond 8 KB among them), by the staged lists (other
# widths, fp32, what the single-launch kernel runs), and a narrow head with 64 candidates that counts
# by the former although the latter kernel runs it
NOALLOC_LIMITS = [((4096, 32000, 16, 2, 10, BF16), 60), ((4096, 32000, 16, 2, 10, 2), 60), ((4096, 32000, 32, 4, 10, BF16), 56),
                  ((4096, 50257, 16, 2, 10, BF16), 39), ((2560, 50257, 48, 3, 20, BF16), 36), ((8192, 32000, 16, 2, 10, BF16), 60),
                  ((5120, 128256, 32, 4, 10, BF16), 15), ((4096, 128256, 32, 4, 10, BF16), 16), ((3584, 152064, 32, 4, 10, BF16), 16),
                  ((1664, 50272, 16, 2, 10, BF16), 51), ((2308, 50272, 16, 2, 10, F32), 51), ((256, 8192, 16, 2, 64, F32), 31)]


@pytest.mark.skipif(torch.cuda.is_available(), reason="the made-up addresses would be launched with")
@pytest.mark.parametrize("shape,most", NOALLOC_LIMITS)
def test_noalloc_takes_the_sizes_it_always_took(shape, most):
    assert noalloc_status(most, *shape) == HIP
    assert noalloc_status(most + 1, *shape) == WORKSPACE


@pytest.mark.skipif(torch.cuda.is_available(), reason="the made-up addresses would be launched with")
def test_noalloc_sizes_of_a_narrow_head_with_many_candidates():
    assert coral.coral_lmhead_path(False, 16, 512, 32000, 16, 2, 64, BF16) == 1
    took = [m for m in range(1, 65) if noalloc_status(m, 512, 32000, 16, 2, 64, BF16) == HIP]
    assert took == [*range(1, 13), *range(16, 61)]       # up to 12 by its lists, from 16 on by the tile path's arrays


# Heads whose calls with fewer tokens take a route with larger arrays: log-probabilities in the
# single launch up to 32 tokens, the general path's tile kernels where the full count has no path.
FEWER = [(36, 256, 152064, 48, 3, 20, F32), (33, 256, 9568, 16, 9, 16, F32), (48, 1024, 128256, 61, 8, 16, BF16),
         (25, 3072, 128256, 16, 5, 10, BF16), (38, 5120, 50272, 300, 3, 1, F32), (64, 2048, 913944, 32, 9, 4, 2),
         (64, 4096, 128256, 64, 8, 16, BF16)]


@pytest.mark.parametrize("M,H,V,G,g,k,dt", FEWER)
def test_a_workspace_serves_fewer_tokens(M, H, V, G, g, k, dt):
    wb = coral.coral_lmhead_workspace_bytes
    have = wb(M, H, V, G, g, k, dt)
    assert all(wb(m, H, V, G, g, k, dt) <= have for m in range(1, M))
    assert all(wb(m, H, V, 0, 0, k, dt) <= have for m in range(1, M + 1))       # the dense head too
    if torch.cuda.is_available():
        return                                         # (the made-up addresses would be launched with)
    c = Call()
    c.off = (np.arange(G + 1, dtype=np.int64) * V // G).astype(np.int32)
    c.gi = coral._GroupIndexStruct(G, c.off.ctypes.data, FAKE + 0x600000, FAKE + 0x700000)
    for m in range(1, M + 1):
        kw = dict(M=m, H=H, V=V, g=g, k=k, dt=dt, ws_bytes=have)
        assert c.grouped(**kw) in (HIP, UNSUPPORTED) and c.dense(**kw) in (HIP, UNSUPPORTED)


def test_log_probabilities_beyond_32_tokens_stay_in_one_launch_where_the_tile_kernels_do_not_fit():
    """The ranking kernel's tables in LDS end at about 660 000 vocabulary rows."""
    lp = coral.coral_lmhead_logprob_path
    assert lp(32, 256, 128256, 32, 2, 8, BF16) == 1 and lp(33, 256, 128256, 32, 2, 8, BF16) == 0
    assert lp(33, 512, 128256, 32, 2, 8, BF16) == 2
    for M in (32, 33, 48):
        assert lp(M, 256, 700_000, 32, 2, 8, BF16) == 1
        assert lp(M, 512, 700_000, 32, 2, 8, BF16) == 1


def test_routes_on_both_sides_of_the_dispatch_rules():
    path, lp = coral.coral_lmhead_path, coral.coral_lmhead_logprob_path
    # rows beyond 8 KB: the single launch with few groups and tokens, more of both with many candidates
    assert path(False, 1, 4616, 128_000, 128, 2, 10, BF16) == 1 and path(False, 1, 4616, 128_100, 300, 2, 10, BF16) == 0
    assert path(False, 6, 4616, 128_000, 80, 2, 10, BF16) == 1 and path(False, 6, 4616, 128_000, 128, 2, 10, BF16) == 0
    assert path(False, 6, 4616, 128_000, 128, 2, 33, BF16) == 1
    assert lp(8, 5888, 42_200, 25, 2, 4, BF16) == 1 and lp(6, 4616, 128_000, 100, 3, 10, BF16) == 0
    assert path(False, 1, 8192, 128_100, 300, 2, 10, BF16) == 1    # the other choice is the matrix-core path
    assert path(False, 6, 5120, 128_256, 48, 2, 10, BF16) == 2     # its blocks fill most of one round
    assert path(False, 6, 5120, 128_256, 32, 2, 10, BF16) == 1     # ... a second one, mostly empty
    # many tokens whose candidates would have to be kept in lists
    assert path(True, 15, 4096, 60_000, 0, 0, 10, BF16) == 1 and path(True, 16, 4096, 60_000, 0, 0, 10, BF16) == 2
    assert path(False, 31, 256, 1_000_000, 4, 2, 10, BF16) == 1 and path(False, 64, 512, 128_256, 4, 2, 10, BF16) == 2
    assert path(False, 62, 232, 104_160, 20, 7, 10, F32) == 0


def test_dense_heads_with_many_tokens_take_the_tile_kernels():
    """Either side of the rule: tokens, rows, storage type."""
    BF16, F32 = coral.CORAL_BF16, coral.CORAL_F32
    path = coral.coral_lmhead_path
    assert path(True, 15, 1024, 38_654, 0, 0, 10, BF16) == 1 and path(True, 16, 1024, 38_654, 0, 0, 10, BF16) == 0
    assert path(True, 16, 1000, 9_000, 0, 0, 1, BF16) == 0 and path(True, 16, 1000, 8_191, 0, 0, 1, BF16) == 1
    assert path(True, 23, 512, 9_000, 0, 0, 1, F32) == 1 and path(True, 24, 512, 9_000, 0, 0, 1, F32) == 0
    # few blocks, a second round for a few of them, fp32 whose rounds take as long as the vector units: the single launch
    assert path(True, 18, 1736, 11_449, 0, 0, 33, BF16) == 1 and path(True, 24, 1736, 32_000, 0, 0, 33, BF16) == 0
    assert path(True, 19, 2320, 33_780, 0, 0, 1, BF16) == 1 and path(True, 19, 2320, 32_700, 0, 0, 1, BF16) == 0
    assert path(True, 26, 944, 33_304, 0, 0, 10, F32) == 1 and path(True, 26, 944, 32_700, 0, 0, 10, F32) == 0
    # the plain form where a workgroup would keep sorted lists, and where the vocabulary is large
    assert path(True, 16, 4096, 60_000, 0, 0, 10, BF16) == 2 and path(True, 8, 1024, 65_536, 0, 0, 10, BF16) == 2


# tokens, H, V, groups, g, k, storage: either side of where the tile kernels take 16-bit grouped heads with many
# tokens; what stays on the single launch measured 0.86 to 0.95 of its speed there
MANY_TOKENS = [((41, 776, 38275, 59, 3, 1, F16), 1), ((40, 520, 10371, 27, 1, 1, BF16), 1), ((40, 520, 10371, 27, 1, 4, BF16), 0),
               ((40, 512, 11353, 18, 1, 1, BF16), 2), ((39, 472, 35451, 27, 2, 1, F16), 1), ((39, 472, 32768, 27, 2, 1, F16), 0),
               ((38, 712, 32295, 29, 2, 2, F16), 1), ((38, 712, 32295, 29, 8, 2, F16), 0), ((37, 488, 125086, 13, 1, 10, BF16), 1),
               ((37, 512, 125086, 13, 1, 10, BF16), 2), ((37, 488, 50000, 13, 1, 10, BF16), 0), ((38, 984, 33128, 33, 4, 10, BF16), 1),
               ((38, 984, 31000, 33, 4, 10, BF16), 0), ((40, 488, 125086, 200, 1, 10, BF16), 0), ((40, 488, 125086, 8, 4, 10, BF16), 0),
               ((50, 776, 38275, 59, 3, 1, F16), 0), ((49, 312, 142728, 24, 2, 8, F16), 1), ((50, 312, 142728, 24, 2, 8, F16), 0)]


@pytest.mark.parametrize("sizes,path", MANY_TOKENS)
def test_route_of_grouped_heads_with_many_tokens(sizes, path):
    assert coral.coral_lmhead_path(False, *sizes) == path


@pytest.mark.parametrize("H,dt", [(4224, BF16), (4352, F16), (4608, BF16), (2112, F32), (2304, F32)])
def test_route_of_rows_of_nine_segments(H, dt):
    """Single launch: dense up to seven tokens; log-probabilities up to eight, and with few tokens a group (6 of 8
    groups: 0.75 of them); grouped by tokens a group.  Whole 512-column chunks in 16 bits: where the matrix-core
    path is the other choice, fewer tokens a group, and no more scores than words for them."""
    chunks = H == 4608
    for M in (1, 4, 7, 8, 9, 11, 12):
        tokens = M * 6 / (8 * (1 - 0.25 ** M))
        path = coral.coral_lmhead_path(False, M, H, 91704, 8, 6, 8, dt)
        assert (path == 1) == (tokens <= (6.0 if chunks else 8.5 if dt == F32 else 7.5))
        assert path in (1, 2 if chunks else 0)
        assert coral.coral_lmhead_path(False, M, H, 91704, 8, 6, 17, dt) == 1
        lp = coral.coral_lmhead_logprob_path(M, H, 91704, 8, 6, 8, dt)
        assert (lp == 1) == (M <= 8 and tokens <= (3.5 if chunks else 8.0 if dt == F32 else 6.0))
        assert (coral.coral_lmhead_path(True, M, H, 24624, 0, 0, 8, dt) == 1) == (M <= (6 if chunks else 7))
        assert (coral.coral_lmhead_path(True, M, H, 16383, 0, 0, 8, dt) == 1) == (M <= 7)
        assert chunks or (coral.coral_lmhead_logprob_path(M, H, 16000, 8, 6, 8, dt) == 1) == (M <= 8)
    assert coral.coral_lmhead_path(False, 14, H, 56000, 8, 7, 64, dt) != 1
    # many tokens a group, blocks of half a round over the compute units, of most of one, of little more and two
    for V, fused in ((16000, True), (30000, False), (40000, True), (60000, False)):
        assert (coral.coral_lmhead_path(False, 14, H, V, 8, 7, 8, dt) == 1) == (fused and not chunks)
    # 4096 scores and more than that
    assert coral.coral_lmhead_path(False, 4, H, 80000, 1024, 3, 17, dt) == 1
    assert coral.coral_lmhead_path(False, 4, H, 80000, 1025, 3, 17, dt) != 1
    # log-probabilities, many candidates beside the matrix-core path: 8 of 24 groups, 9 of 24 groups, one token
    for M in (1, 3):
        assert coral.coral_lmhead_logprob_path(M, H, 10896, 24, 8, 64, dt) == 1
        assert (coral.coral_lmhead_logprob_path(M, H, 10896, 24, 9, 64, dt) == 1) == (not chunks)


def test_route_of_longer_rows_by_tokens_a_group():
    """More groups than the own gate was taken for: up to ten tokens a group."""
    assert coral.coral_lmhead_path(False, 12, 2816, 111132, 126, 100, 1, F32) == 1
    assert coral.coral_lmhead_path(False, 12, 2816, 111132, 126, 109, 1, F32) == 0


@pytest.mark.parametrize("H", [4224, 4608, 4616, 4736, 5120, 8192])
def test_no_own_gate_with_log_probabilities_beyond_8_kb(H):
    """16 bits, four tokens and more, more scores than can be shared: the single launch has no form for it."""
    for M in (4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 16, 32, 64):
        for G in sorted({4096 // M + 1, 4096 // M + 9, 256, 400, 512, 513, 1024}):
            for k in (1, 10, 33, 50, 64):
                for g in {1, 3, max(1, 64 // M)}:
                    assert M * G <= 4096 or coral.coral_lmhead_logprob_path(M, H, 150000, G, g, k, BF16) != 1
