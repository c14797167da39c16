"""Launches of one epoch that could run beside a sweep's plain stores: on another
stream while the sweep's own records a graph, from a graph recorded earlier, on
a stream whose handle a destroyed one had.  Both kernels start at one event, so
that they overlap unless one waits; a lost update then loses races.  And calls
that do not wait on the host."""
import ctypes
import time

import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

SIDE = 2048
CELLS = np.arange(3, SIDE * SIDE, 16)


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2401_04701_amd import hr
    torch.cuda.set_device(0)
    return torch, hr


class Hip:
    """The runtime that the process has loaded."""

    def __init__(self):
        with open("/proc/self/maps") as f:
            path = next(w for line in f for w in line.split() if "libamdhip64.so" in w)
        self.lib = ctypes.CDLL(path)

    def __call__(self, name, *args):
        st = getattr(self.lib, name)(*args)
        assert st == 0, (name, st)

    def begin(self, stream):
        self("hipStreamBeginCapture", ctypes.c_void_p(stream), 1)      # thread-local mode

    def end(self, stream):
        g = ctypes.c_void_p()
        self("hipStreamEndCapture", ctypes.c_void_p(stream), ctypes.byref(g))
        return g


def writes_launch():
    """A program whose threads write every sixteenth cell of region 1, from the
    last cell on: nearly all in another block than the sweep's."""
    threads, blocks = 256, 256
    n = len(CELLS)
    off = np.linspace(0, n, threads * blocks + 1).astype(np.int32)
    ops = (CELLS[::-1] | 1 << 24 | 1 << 27).astype(np.uint32)
    return si.Launch(blocks=blocks, threads=threads, scope=np.zeros(1, np.uint8),
                     wave_mask=np.zeros(1, np.uint64), op_off=off, ops=ops)


def same_block():
    """Cells that the sweep and the program write in a block of one number: a
    block's clock stands at 1 at the sweep's writes and at 0 at the program's,
    so a barrier orders the two."""
    y, x = CELLS // SIDE, CELLS % SIDE
    place = np.arange(len(CELLS) - 1, -1, -1)          # position of each cell in the ops
    return set(CELLS[y // 16 * (SIDE // 16) + x // 16 == place * 256 // len(CELLS)].tolist())


class Job:
    def __init__(self, torch, hr):
        self.torch, self.hr, self.hip = torch, hr, Hip()
        self.prog = hr.DeviceProgram(writes_launch())
        self.u = [torch.rand((SIDE, SIDE), device="cuda"), torch.zeros((SIDE, SIDE), device="cuda")]
        self.want = set(CELLS.tolist()) - same_block()
        assert len(self.want) > 0.99 * len(CELLS)
        self.ctx = hr.Context(ring_capacity=1 << 20)
        self.regs = [self.ctx.shadow_alloc(x) for x in self.u]
        torch.cuda.synchronize()

    def sweep(self, stream=None):
        self.ctx.jacobi_check(*self.regs, *self.u, None, stream=stream)

    def writes(self, stream=None):
        self.ctx.program_check(self.prog, self.regs, 0, stream=stream)

    def gate(self, first, *others):
        """Streams that go on together, some milliseconds from now."""
        ev = self.torch.cuda.Event()
        with self.torch.cuda.stream(first):
            self.torch.cuda._sleep(20_000_000)
            ev.record()
        for s in others:
            s.wait_event(ev)

    def check(self):
        self.torch.cuda.synchronize()
        got = {k[3] for k in self.ctx.flagged()}
        assert self.ctx.status == 0 and len(got) == len(self.want) and got == self.want


@pytest.mark.parametrize("home", [True, False])
def test_the_sweeps_stream_records(env, home):
    """The sweep's stream begins to record behind it; the writes go elsewhere."""
    torch, hr = env
    print("[case] epoch waits, recording stream, home", home, flush=True)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a if home else torch.cuda.Stream()):
        j = Job(torch, hr)
    for _ in range(3):
        j.ctx.reset(stream=b)
        torch.cuda.synchronize()
        j.gate(a, b)
        j.sweep(a)
        j.hip.begin(a.cuda_stream)
        j.writes(b)
        j.hip("hipGraphDestroy", j.hip.end(a.cuda_stream))
        j.check()
    j.ctx.close()


@pytest.mark.parametrize("recorded_on", ["a", "b"])
def test_a_graph_replayed_beside_the_sweep(env, recorded_on):
    """The writes are recorded behind the sweep and replayed at once elsewhere."""
    torch, hr = env
    print("[case] epoch waits, graph at once, recorded on", recorded_on, flush=True)
    s = {"a": torch.cuda.Stream(), "b": torch.cuda.Stream()}
    c = torch.cuda.Stream()
    for _ in range(3):                       # a context each: its first recording
        with torch.cuda.stream(s["a"]):
            j = Job(torch, hr)
        j.gate(s["a"], c)
        j.sweep(s["a"])
        r = s[recorded_on]
        j.hip.begin(r.cuda_stream)
        j.writes(r)
        g, ex = j.hip.end(r.cuda_stream), ctypes.c_void_p()
        j.hip("hipGraphInstantiate", ctypes.byref(ex), g, None, None, ctypes.c_size_t(0))
        j.hip("hipGraphLaunch", ex, ctypes.c_void_p(c.cuda_stream))
        j.check()
        j.hip("hipGraphExecDestroy", ex)
        j.hip("hipGraphDestroy", g)
        j.ctx.close()


def test_a_graph_of_an_earlier_epoch(env):
    """A graph recorded once is replayed beside later jobs' sweeps."""
    torch, hr = env
    print("[case] epoch waits, earlier graph", flush=True)
    a, c = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        j = Job(torch, hr)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=c):
        j.writes()
    for _ in range(3):
        j.ctx.reset(stream=a)
        torch.cuda.synchronize()
        j.gate(a, c)
        with torch.cuda.stream(c):
            g.replay()
        j.sweep(a)
        j.check()
    j.ctx.close()


def test_a_destroyed_streams_handle(env):
    """The sweep's stream is destroyed at once; a new one may have its handle."""
    torch, hr = env
    print("[case] epoch waits, destroyed stream", flush=True)
    j = Job(torch, hr)

    def create():
        s = ctypes.c_void_p()
        j.hip("hipStreamCreateWithFlags", ctypes.byref(s), 1)
        return s

    for _ in range(4):
        j.ctx.reset()
        torch.cuda.synchronize()
        x = create()
        j.gate(torch.cuda.ExternalStream(x.value))
        j.sweep(x.value)
        j.hip("hipStreamDestroy", x)
        y = create()
        j.writes(y.value)
        j.check()
        j.hip("hipStreamDestroy", y)
    j.ctx.close()


def test_a_sweep_on_a_second_stream_returns_at_once(env):
    torch, hr = env
    print("[case] epoch waits, asynchronous sweep", flush=True)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        j = Job(torch, hr)

    def both(busy):
        with torch.cuda.stream(a):
            torch.cuda._sleep(busy)
        j.sweep(a)
        j.sweep(b)
        j.ctx.kernel_end(stream=b)             # one epoch on both streams

    both(1000)
    torch.cuda.synchronize()
    t = time.perf_counter()
    both(400_000_000)
    called = time.perf_counter() - t
    torch.cuda.synchronize()
    done = time.perf_counter() - t
    assert done > 0.02 and called < done / 3
    j.ctx.close()


def test_label_propagation_on_a_second_stream_returns_at_once(env):
    """One job after the other on two streams, and both streams in one job."""
    torch, hr = env
    print("[case] epoch waits, asynchronous label propagation", flush=True)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        ctx = hr.Context()
        n = 4000
        rp = torch.arange(n + 1, dtype=torch.int32, device="cuda")
        col = torch.arange(1, n + 1, dtype=torch.int32, device="cuda") % n
        mask = torch.zeros(n, dtype=torch.uint8, device="cuda")
        label = torch.arange(n, dtype=torch.int32, device="cuda")
        r = ctx.shadow_alloc(label)

    def sweep(s):
        ctx.labelprop_check(r, label, rp, col, mask, stream=s)
        ctx.kernel_end(stream=s)

    def jobs(busy):
        with torch.cuda.stream(a):
            torch.cuda._sleep(busy)
        for s in (a, b, a):
            ctx.reset(stream=s)
            sweep(s)
        sweep(b)

    jobs(1000)
    torch.cuda.synchronize()
    t = time.perf_counter()
    jobs(400_000_000)
    called = time.perf_counter() - t
    torch.cuda.synchronize()
    done = time.perf_counter() - t
    assert done > 0.02 and called < done / 3
    ctx.close()
