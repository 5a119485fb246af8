"""The host side of headkv_assign_budgets on the CPU: csrc/headkv_abi.cpp built
against tests/host/fake_hip.cpp, which stands in for the HIP runtime and the
kernels and counts pinned allocations and frees."""
import ctypes
import os
import shutil
import subprocess
import threading

import numpy as np
import pytest

from paper_2605_20600_amd import binding as B
from paper_2605_20600_amd.build import CSRC

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
N = 4500  # num_visual


class Counts(ctypes.Structure):
    _fields_ = [(n, ctypes.c_long) for n in ("mallocs", "frees", "unsafe_calls", "copies",
                                             "live_buffers", "live_bytes", "max_live")]


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    lib = tmp_path_factory.mktemp("fake") / "libheadkv_fake.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    os.path.join(HERE, "host", "fake_hip.cpp"),
                    os.path.join(CSRC, "headkv_abi.cpp"), "-Wl,-z,defs", "-o", str(lib)],
                   check=True)
    return lib


@pytest.fixture
def fake(built, tmp_path, monkeypatch):
    # a copy of its own: the library keeps its pinned buffers until the process ends
    path = tmp_path / "libheadkv.so"
    shutil.copy(built, path)
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "LIB_PATH", str(path))
    lib = B.load()
    lib.fake_counts.restype = Counts
    lib.fake_last_host.restype = ctypes.c_void_p
    return lib


def _buffer(n):
    a = np.zeros(n + 256, np.uint8)
    return a[-a.ctypes.data % 256:][:n]


class Handle:
    """A one-layer handle at its grouping step (group_threshold 1)."""

    def __init__(self, batch, strategy=B.HEADKV_ATTN_VARLEN, heads=8, d=64):
        self.cfg = B.HeadKVConfig(
            batch=batch, num_layers=1, num_heads=heads, head_dim=d, prefix_len=0, row_len=10,
            num_visual=N, recent_len=20, local_window=20, period=1, group_threshold=1,
            budget_mode=B.HEADKV_BUDGET_OVERRIDE, rho_num=1, rho_den=2, rs_num=1, rs_den=2,
            attn_strategy=strategy, score_mode=0, cfg_pairs=0, tau=0.9)
        self.BH = heads * batch
        self.sizes = B.headkv_plan(self.cfg)
        self.dense, self.meta, self.ws = (_buffer(n) for n in self.sizes)
        self.h = B.headkv_create(self.cfg, [self.dense.ctypes.data], [self.meta.ctypes.data],
                                 self.ws.ctypes.data)
        B.headkv_prefill(self.h, 0, None, None)
        self.row = _buffer(self.BH * d * 2)
        B.headkv_append_and_evict(self.h, 0, 0, *(3 * [self.row.ctypes.data]))
        self.labels = np.zeros(self.BH, np.uint8)
        self.budgets = np.zeros(self.BH, np.int32)
        rng = np.random.default_rng(batch)
        self.override = rng.integers(1, N + 1, self.BH).astype(np.int32)

    def size(self):
        """The sizing call: (status, bytes needed)."""
        return B.headkv_assign_budgets(self.h, 0, self.labels.ctypes.data,
                                       self.override.ctypes.data, self.budgets.ctypes.data,
                                       None, 0)

    def assign(self):
        """The whole call, into a segment buffer that the fake kernels do not touch."""
        st, need = B.headkv_assign_budgets(self.h, 0, self.labels.ctypes.data,
                                           self.override.ctypes.data, self.budgets.ctypes.data,
                                           0x7F0000000000, 1 << 62)
        assert st == B.HEADKV_OK, B.headkv_last_error()
        self.check_tables(need)

    def check_tables(self, need):
        BH, at = self.BH, [0]

        def take(dtype, n):
            a = self.meta[at[0]:at[0] + n * np.dtype(dtype).itemsize].view(dtype)
            at[0] = (at[0] + a.nbytes + 255) // 256 * 256
            return a

        seg_off, cap = take(np.int64, BH), take(np.int32, BH)
        for _ in range(2):  # lengths, budgets
            take(np.int32, BH)
        take(np.int32, BH)  # n*
        take(np.int32, BH)  # labels
        order = take(np.int32, BH)
        # room for every head at its largest, in passes of 256 threads
        d = self.cfg.head_dim
        tokens = 256 // (d // 8) * 8
        items = take(np.uint32, BH * ((N + 1 + tokens - 1) // tokens))
        item_start = take(np.int32, BH + 1)
        want_cap = np.minimum(self.override + 1, N)
        assert (self.budgets == self.override).all() and (cap == want_cap).all()
        seg = (2 * want_cap.astype(np.int64) * d * 2 + want_cap * 4 + 255) // 256 * 256
        assert need == seg.sum() and (seg_off == np.cumsum(seg) - seg).all()
        if self.cfg.attn_strategy == B.HEADKV_ATTN_GROUPED:
            assert (order == np.argsort(self.override & 1, kind="stable")).all()
        else:
            assert (order == np.argsort(-want_cap, kind="stable")).all()
        n = np.diff(item_start)
        assert item_start[0] == 0 and (n >= 1).all()
        head = np.repeat(np.arange(BH), n)
        chunk = np.arange(item_start[-1]) - np.repeat(item_start[:-1], n)
        assert (items[:item_start[-1]] == head * 256 + chunk).all()


def test_growing_handles_pin_once(fake):
    # handles whose tables need ever more room: after the first call every one
    # finds a kept buffer that is large enough
    handles = [Handle(batch) for batch in (64, 128, 256, 384, 512, 640, 768)]
    for h in handles:
        h.size()
    before = fake.fake_counts().mallocs
    for _ in range(3):
        for h in handles:
            assert h.size()[0] == B.HEADKV_ERR_CAPACITY
    c = fake.fake_counts()
    assert (c.mallocs - before, c.frees) == (0, 0)
    for h in handles:
        h.assign()


@pytest.mark.parametrize("strategy", [B.HEADKV_ATTN_VARLEN, B.HEADKV_ATTN_GROUPED])
@pytest.mark.parametrize("batch,copies", [
    (256, 0),            # 2,048 heads: everything through pinned memory
    (2048, 5),           # 16,384: the five tables do not fit
    (131072 // 8 + 1, 7)])  # the budgets and labels neither
def test_large_tables_are_not_pinned_for_the_call(fake, batch, copies, strategy):
    h = Handle(batch, strategy)
    h.size()
    before = fake.fake_counts()
    for _ in range(3):
        assert h.size()[0] == B.HEADKV_ERR_CAPACITY
    c = fake.fake_counts()
    assert (c.mallocs, c.frees) == (before.mallocs, 0)
    h.assign()
    d = fake.fake_counts()
    assert (d.mallocs, d.frees, d.copies - c.copies) == (before.mallocs, 0, copies)
    assert d.live_bytes <= 4 << 20


def test_calls_at_once_free_nothing(fake):
    # six calls that hold their buffers at the same time: nothing is freed (a
    # free waits for the whole device, and is refused while another thread
    # captures a graph), and the calls beyond the four buffers copy
    n = 6
    handles = [Handle(64) for _ in range(n)]
    all_in = threading.Barrier(n)
    hook = ctypes.CFUNCTYPE(None)(lambda: all_in.wait(30) and None)
    for _ in range(3):
        fake.fake_on_budgets(hook)
        got = [None] * n
        threads = [threading.Thread(target=lambda i=i: got.__setitem__(i, handles[i].size()))
                   for i in range(n)]
        for t in threads:
            t.start()
        for t in threads:
            t.join(60)
        fake.fake_on_budgets(ctypes.CFUNCTYPE(None)())
        assert [g[0] for g in got] == n * [B.HEADKV_ERR_CAPACITY]
    for h in handles:
        h.assign()
    c = fake.fake_counts()
    assert (c.unsafe_calls, c.frees, c.mallocs, c.max_live) == (0, 0, 4, 4)


@pytest.mark.parametrize("waits", [1, 2])
def test_buffer_of_a_stream_not_waited_for_is_not_used_again(fake, waits):
    # a stream that cannot be waited for (one that captures, for instance) may
    # still run the kernel that writes the buffer
    h = Handle(64)
    fake.fake_fail_wait(waits)  # the one for the budgets, or the one for the move
    with pytest.raises(B.HeadKVError) as e:
        h.assign()
    assert e.value.status == B.HEADKV_ERR_HIP
    lost = fake.fake_last_host()
    assert lost
    g = Handle(64)
    for _ in range(3):
        assert g.size()[0] == B.HEADKV_ERR_CAPACITY
        assert fake.fake_last_host() != lost
    g.assign()
    assert fake.fake_counts().frees == 0


def test_without_pinned_memory(fake):
    # no pinned memory to be had: the call copies, and pins once there is
    h = Handle(64)
    fake.fake_pin_fails(1)
    assert h.size()[0] == B.HEADKV_ERR_CAPACITY
    h.assign()
    assert fake.fake_counts().copies == 2 + 7
    fake.fake_pin_fails(0)
    Handle(64).assign()
    c = fake.fake_counts()
    assert (c.copies, c.live_buffers) == (2 + 7, 1)


@pytest.mark.parametrize("heads,tokens,d,plan", [
    # tokens of the largest head and of the others; threads, tokens per row, chunks
    (4, (4501, 4501), 128, (256, 8, 4 * 36)),     # at most one chunk per compute unit
    (64, (512, 512), 128, (256, 8, 256)),
    (64, (513, 512), 128, (512, 8, 65 * 2 - 1)),  # 257 of 128 tokens
    (128, (513, 512), 128, (1024, 8, 129)),
    (200, (560, 560), 128, (1024, 9, 200)),       # one wide chunk each, two ordinary ones
    (110, (1100, 1100), 128, (1024, 9, 220)),
    (110, (2150, 2150), 64, (1024, 9, 220)),
    (250, (520, 511), 64, (512, 8, 251)),
    (160, (600, 600), 128, (512, 8, 480))])       # more than one per unit at every size
def test_chunk_pass_rule(fake, heads, tokens, d, plan):
    h = Handle(1, heads=heads, d=d)
    # a table is cut for budget + period + the appended token
    h.override[:] = tokens[1] - 2
    h.override[0] = tokens[0] - 2
    h.assign()
    B.headkv_decode_attn(h.h, 0, h.row.ctypes.data, h.row.ctypes.data)
    tpr, items = ctypes.c_int(), ctypes.c_int()
    threads = fake.fake_plan(ctypes.byref(tpr), ctypes.byref(items))
    assert (threads, tpr.value, items.value) == plan
