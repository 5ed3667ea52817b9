"""What the host code plans, launches and copies, checked without a GPU: the
library's own csrc/pced_api.cpp over recording stand-ins for the HIP runtime and
the kernel launchers (tests/host_path.cpp). Device addresses are never read."""
import ctypes
import os
import subprocess

import pytest

from paper_2601_08670_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_08670_amd", "csrc")
DEVICE = 1 << 46  # addresses from here on count as device memory
CAPACITY, HIPERR = 2, 3


@pytest.fixture(scope="session")
def host(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_path") / "host_path.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                    os.path.join(ROOT, "tests", "host_path.cpp"), os.path.join(CSRC, "pced_api.cpp"),
                    "-Wl,-Bsymbolic", "-Wl,--no-undefined", "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.rec_name.restype = ctypes.c_char_p
    lib.rec_value.restype = ctypes.c_long
    lib.pced_workspace_bytes.restype = ctypes.c_size_t
    lib.pced_last_error.restype = ctypes.c_char_p
    return lib


class Batch:
    """A context with one loaded query; calls return the status."""

    def __init__(self, lib, lens, reserve, src=DEVICE, **kw):
        cfg = dict(n_layers=1, n_q_heads=32, n_kv_heads=8, head_dim=128, vocab=1000, dtype="bf16", max_queries=1,
                   max_seqs=len(lens), max_pages=sum(-(-(n + reserve) // 16) for n in lens),
                   max_pages_per_seq=max(-(-(n + reserve) // 16) for n in lens))
        cfg.update(kw)
        self.lib, self.lens, self.layers = lib, lens, cfg["n_layers"]
        self.cfg = _lib.make_config(**cfg)
        self.ctx = ctypes.c_void_p()
        ws = lib.pced_workspace_bytes(ctypes.byref(self.cfg))
        assert lib.pced_create(ctypes.byref(self.cfg), ctypes.c_void_p(DEVICE), ctypes.c_size_t(ws),
                               ctypes.byref(self.ctx)) == 0, self.error()
        self.status = self.load(reserve, src)

    def load(self, reserve, src=DEVICE):
        S, p = len(self.lens), ctypes.c_void_p(DEVICE + (1 << 40))
        ptrs = (ctypes.c_void_p * S)(*[src] * S)
        self.lib.rec_clear()
        return self.lib.pced_load_caches(self.ctx, 1, (ctypes.c_int32 * 1)(S - 1), (ctypes.c_int32 * S)(*self.lens),
                                         ptrs, ptrs, p, p, None, reserve, (ctypes.c_float * (S - 1))(*[0.5] * (S - 1)),
                                         ctypes.c_float(2.5), None, None)

    def prefill(self, n_tokens):
        self.lib.rec_clear()
        p = ctypes.c_void_p(DEVICE)
        return self.lib.pced_model_prefill(self.ctx, p, n_tokens, p, None)

    def step(self):
        self.lib.rec_clear()
        p = ctypes.c_void_p(DEVICE)
        return self.lib.pced_step(self.ctx, p, p, p, p, p, None, None)

    def calls(self, name):
        return [[self.lib.rec_value(i, j) for j in range(8)] for i in range(self.lib.rec_count())
                if self.lib.rec_name(i).decode() == name]

    def error(self):
        return self.lib.pced_last_error().decode()

    def __del__(self):
        if self.ctx:
            self.lib.pced_destroy(self.ctx)


# attention launches: first layer, layers, chunks, prefill, tokens per group, tokens, partial states per sequence, sequences
LAYER, LAYERS, CHUNKS, PREFILL, TQ, TOKENS, PARTS, SEQS = range(8)


@pytest.mark.parametrize("short,n_short,long,suffix", [
    (16, 75, 8192, 16), (16, 70, 6000, 32), (24, 55, 12288, 20), (1, 100, 30000, 7), (16, 8, 100000, 16),
])
def test_prefill_takes_many_short_caches_beside_a_long_one(host, short, n_short, long, suffix):
    # the partial states that the longest chunks (64 pages) need do not depend on how short the others are
    b = Batch(host, [16] + [short] * n_short + [long], suffix, ffn_dim=512)
    assert b.status == 0 and b.prefill(suffix) == 0, b.error()


@pytest.mark.parametrize("n,long,suffix,tq", [
    (33, 10000, 64, 8),   # the longest chunks take most of the partial-state slots with groups of any size
    (33, 14000, 60, 8), (20, 14000, 100, 8),
    (2, 3000, 64, 8),     # (a plan for the whole chip)
])
def test_prefill_groups_stay_full_where_the_longest_chunks_fit(host, n, long, suffix, tq):
    b = Batch(host, [16] * n + [long], suffix, ffn_dim=512)
    assert b.status == 0 and b.prefill(suffix) == 0, b.error()
    a = b.calls("attn")[0]
    assert a[TQ] == tq and a[TOKENS] == suffix, a


def test_prefill_groups_shrink_only_to_save_padding(host):
    # 9 tokens as two groups of 5 are 10 columns; as 9 groups of one they are 9
    b = Batch(host, [16] * 230 + [16 * 64 * 15], 9, ffn_dim=512)
    assert b.status == 0 and b.prefill(9) == 0, b.error()
    a = b.calls("attn")[0]
    assert 231 * 9 * a[PARTS] <= 2 * 2304 * 8 < 231 * 10 * a[PARTS] and a[TQ] in (1, 3), a
    assert Batch(host, [16] * 230 + [16 * 64 * 20], 9, ffn_dim=512).prefill(9) == CAPACITY


@pytest.mark.parametrize("layers,lens,cap", [
    (32, [64] + [1500] * 32, 4),   # more pages than 64 per chunk: a launch per layer, as many chunks as it needs
    (32, [64] + [1500] * 32, 256), (32, [64] + [1500] * 32, 100), (5, [16] + [90] * 3, 2), (7, [16] + [90] * 8, 4),
    (32, [16] + [700] * 4, 9), (1, [16] + [700] * 4, 3), (32, [64] + [1500] * 32, 0), (5, [16] + [90] * 3, 0),
])
def test_step_launches_keep_to_the_chunk_cap(host, layers, lens, cap):
    b = Batch(host, lens, 2, n_layers=layers, max_attn_chunks=cap)
    assert b.status == 0 and b.step() == 0, b.error()
    at, nxt = b.calls("attn"), 0
    for a in at:  # every layer once, in order
        assert a[LAYER] == nxt and a[LAYERS] >= 1
        nxt += a[LAYERS]
        assert not cap or a[LAYERS] == 1 or a[LAYERS] * a[CHUNKS] <= cap, a
    assert nxt == layers
    pages = sum(-(-(n + 1) // 16) for n in lens)
    if cap:
        assert at[0][CHUNKS] <= max(cap, -(-pages // 64), pages // 2), at[0]
    else:
        assert len(at) == 1


@pytest.mark.parametrize("suffix,cap", [(9, 4), (64, 8), (64, 100), (1, 3)])
def test_prefill_launch_keeps_to_the_chunk_cap(host, suffix, cap):
    lens = [16] + [800] * 8
    b = Batch(host, lens, suffix, ffn_dim=512, max_attn_chunks=cap)
    assert b.status == 0 and b.prefill(suffix) == 0, b.error()
    groups = -(-suffix // b.calls("attn")[0][TQ])
    pages = sum(-(-(n + suffix) // 16) for n in lens)
    assert b.calls("attn")[0][CHUNKS] * groups <= max(cap, groups * -(-pages // 64))


@pytest.mark.parametrize("call,nth", [("copy_in", 3), ("copy_in", 4), ("load", 1), ("load", 2)])
def test_failing_host_load_waits_for_its_copies(host, call, nth):
    # (the first copy is the metadata; then K, V and a launch per sequence)
    b = Batch(host, [40, 50, 60], 0)
    host.rec_fail(call.encode(), nth)
    assert b.load(0, src=4096) == HIPERR
    host.rec_fail(b"", 0)
    assert host.rec_name(host.rec_count() - 1) == b"synchronize"
    assert b.load(0, src=4096) == 0 and len(b.calls("synchronize")) == 1 and len(b.calls("copy_in")) == 7


def _workspace(host, **kw):
    c = dict(n_layers=32, n_q_heads=32, n_kv_heads=8, head_dim=128, vocab=1000, dtype="bf16", max_queries=1,
             max_seqs=33, max_pages=33 * 130, max_pages_per_seq=130)
    c.update(kw)
    return host.pced_workspace_bytes(ctypes.byref(_lib.make_config(**c)))


def test_attention_plan_is_sized_by_pages(host):
    # a page more per sequence costs the rows' and the sequences' page tables (4 bytes a row) and room for
    # partial states, but no plan entries (520 bytes each) per suffix row
    grow = _workspace(host, ffn_dim=512, max_pages_per_seq=131) - _workspace(host, ffn_dim=512)
    plain = _workspace(host, max_pages_per_seq=131) - _workspace(host)
    assert grow - plain <= 4 * (2304 + 33) + 131 * 16 * 64 * 8 + 8 * 256


def test_workspace_holds_one_layer_output(host):
    # a layer more: pced_generate's q, k and v rows (12288 bytes a sequence), room for partial states and for
    # staging a cache from host memory, but no copy of the layer's output (8192 bytes a sequence)
    short = dict(max_pages=33, max_pages_per_seq=1)
    grow = _workspace(host, n_layers=33, **short) - _workspace(host, n_layers=32, **short)
    assert grow <= 33 * 12288 + 33 * 8 * (2048 + 64) + 2 * 16 * 8 * 128 * 2 + 33 * 4096


def test_host_caches_are_staged_in_the_partial_states_region(host):
    # K and V of 130 pages x 32 layers: 130 MiB, moved in pieces of 2 x 32 MiB; the partial states take 34 MiB
    shape = dict(n_q_heads=8, max_seqs=2, max_pages=260)
    assert 64 << 20 < _workspace(host, **shape) < 80 << 20
    b = Batch(host, [2000, 16, 40], 4, n_layers=32, src=4096)
    assert b.status == 0, b.error()
    copies, ws = b.calls("copy_in")[1:], host.pced_workspace_bytes(ctypes.byref(b.cfg))
    assert sum(c[0] for c in copies) == 2 * 2056 * 32 * 8 * 128 * 2 and max(c[0] for c in copies) <= 32 << 20
    assert all(DEVICE <= c[1] and c[1] + c[0] <= DEVICE + ws for c in copies)


@pytest.mark.parametrize("layers,lens,kw", [
    (32, [64] + [1024] * 8, {}), (32, [64] + [500 + 50 * i for i in range(32)], {}), (32, [16] + [30] * 64, {}),
    (16, [16, 20000] + [40] * 6, {}), (2, [64] + [2000] * 32, {}), (32, [64] * 5, dict(dtype="f32")),
    (32, [16] + [300] * 16, dict(n_q_heads=16, n_kv_heads=16, head_dim=64)),
])
def test_partial_states_of_all_layers_fit(host, layers, lens, kw):
    b = Batch(host, lens, 4, n_layers=layers, **kw)
    assert b.status == 0 and b.step() == 0, b.error()
    assert [a[LAYERS] for a in b.calls("attn")] == [layers]


def test_partial_states_take_no_more_than_a_usual_plan(host):
    # 9 sequences x 20 pages x 32 layers: 32 MiB of staging, where the worst plan of all layers is 94 MiB
    assert _workspace(host, max_seqs=9, max_pages=180, max_pages_per_seq=20) < 64 << 20
