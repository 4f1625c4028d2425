"""The Python binding on the host: what it hands to the library."""
import ctypes

import pytest
import torch

from paper_2609_33570_amd import hilore

FIELDS = [name for name, _ in hilore.hilore_unit_desc._fields_]


class Longer(hilore.hilore_unit_desc):
    _fields_ = [("tag", ctypes.c_int64)]


class Renamed(hilore.hilore_unit_desc):
    pass


def values(i):
    return tuple((1 << 20) + 4096 * i + 256 * k for k in range(6)) + (10 + i, 128 * (i + 1), 128 * (i + 2))


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 17])
@pytest.mark.parametrize("make", [
    lambda i: hilore.hilore_unit_desc(*values(i)),
    lambda i: Longer(*values(i), 7),
    lambda i: Renamed(*values(i)),
    values,
    lambda i: (hilore.hilore_unit_desc(*values(i)), Longer(*values(i), 7), values(i))[i % 3],
], ids=["plain", "longer", "renamed", "tuple", "mixed"])
def test_descriptor_array(make, n):
    """Every form of descriptor that a ctypes array takes arrives unchanged, in any number."""
    arr, count = hilore._desc_array([make(i) for i in range(n)])
    assert count == n and ctypes.sizeof(arr) == 72 * max(1, n)
    for i in range(n):
        assert tuple(getattr(arr[i], f) for f in FIELDS) == values(i)


@pytest.mark.parametrize("n", [1, 5])
def test_descriptor_array_refuses_other_types(n):
    with pytest.raises(TypeError):
        hilore._desc_array([ctypes.c_int64(3)] * n)


# --------------------------------------------- memory of the split weight gradient --
NEED, OWN_STREAM, SCRATCH = 1 << 21, 0x5150, 1 << 30


class FakeTensor:
    """What the binding asks of a device tensor."""

    is_cuda = True

    def __init__(self, device=0):
        self.device = torch.device("cuda", device)

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 1 << 20


class FakeLibrary:
    """Records which entry point the binding calls and with what memory."""

    def __init__(self, capturing, need):
        self.capturing, self.need, self.calls = capturing, need, []

    def hilore_wgrad_workspace_bytes(self, K, M, N):
        return self.need

    def hipStreamIsCapturing(self, stream, status):
        status._obj.value = 1 if self.capturing else 0
        return 0

    def hilore_dequant_wgrad(self, *args):
        self.calls.append(("unsplit", None, args[10]))
        return hilore.HILORE_OK if args[5] else hilore.HILORE_ERR_INVALID_ARG

    def hilore_dequant_wgrad_ws(self, *args):
        self.calls.append(("split", args[10:12], args[12]))
        return hilore.HILORE_OK

    def hilore_status_string(self, status):
        return b"status"


@pytest.fixture
def fake(monkeypatch):
    """hilore_dequant_wgrad on a host without a GPU: the library and torch's allocator faked."""
    state = {"live": {}, "taken": []}

    def alloc(size, device=None, stream=None):
        if size >= state.get("limit", 1 << 40):
            raise torch.cuda.OutOfMemoryError("no memory left")
        device = torch.device(device).index if not isinstance(device, int) else device
        state["taken"].append((size, device, stream))
        p = SCRATCH + len(state["taken"]) * 4096
        state["live"][p] = size
        return p

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", alloc)
    monkeypatch.setattr(torch.cuda, "caching_allocator_delete", lambda p: state["live"].pop(p))

    class Tensor:
        def __init__(self, n, dtype, device):
            self.p = alloc(n, device, OWN_STREAM)

        def data_ptr(self):
            return self.p

        def __del__(self):
            if hasattr(self, "p"):
                state["live"].pop(self.p)

    monkeypatch.setattr(torch, "empty", Tensor)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: OWN_STREAM, raising=False)
    monkeypatch.setattr(torch.cuda, "memory_snapshot", lambda: [
        {"address": SCRATCH, "total_size": 1 << 21, "segment_pool_id": state.get("pool", (0, 0))}])

    def call(capturing=False, need=NEED, dw=FakeTensor(), **kw):
        lib = FakeLibrary(capturing, need)
        monkeypatch.setattr(hilore, "load", lambda: lib)
        x = FakeTensor()
        try:
            hilore.hilore_dequant_wgrad(x, x, 1, 128, x, dw, 16384, 3584, 512, **kw)
        finally:
            assert not state["live"], "memory kept after the call"
        (entry,) = lib.calls
        return entry

    call.state = state
    return call


@pytest.mark.parametrize("kw,stream", [({}, OWN_STREAM), ({"stream": 77}, 77)], ids=["current", "explicit"])
def test_wgrad_scratch_in_stream_order(fake, kw, stream):
    """Taken for the call's stream, handed over whole, given back when the call is enqueued."""
    name, (ptr, nbytes), handle = fake(**kw)
    assert name == "split" and nbytes == NEED and ptr > SCRATCH and handle == stream
    assert fake.state["taken"] == [(NEED, 0, stream)]
    assert fake(need=0, **kw) == ("unsplit", None, stream) and len(fake.state["taken"]) == 1


@pytest.mark.parametrize("kw", [{}, {"stream": 77}], ids=["current", "explicit"])
def test_wgrad_under_capture(fake, kw):
    """A graph keeps writing a captured call's memory: it may come from a graph's own pool
    only, and without one (a capture that torch has not begun) the call takes none."""
    fake.state["pool"] = (0, 0)
    assert fake(capturing=True, **kw)[0] == "unsplit"
    fake.state["pool"] = (3, 0)
    assert fake(capturing=True, **kw)[0] == "split"


def test_wgrad_scratch_of_another_device(fake):
    """The current stream orders the reuse of memory of its own device."""
    assert fake(dw=FakeTensor(1))[0] == "split"
    assert fake.state["taken"] == [(NEED, 0, OWN_STREAM)]
    assert fake(dw=FakeTensor(1), stream=77)[0] == "split"
    assert fake.state["taken"][1:] == [(NEED, 1, 77)]


def test_wgrad_without_output(fake):
    """A call without dw is the library's to refuse."""
    with pytest.raises(hilore.HiloreError) as e:
        fake(dw=None, stream=0)
    assert e.value.status == hilore.HILORE_ERR_INVALID_ARG and not fake.state["taken"]


@pytest.mark.parametrize("kw", [{}, {"stream": 77}], ids=["current", "explicit"])
def test_wgrad_out_of_memory(fake, kw):
    """Runs unsplit, whose rounding differs, and says so."""
    fake.state["limit"] = NEED
    with pytest.warns(RuntimeWarning, match="unsplit"):
        assert fake(**kw)[0] == "unsplit"


def test_wgrad_on_the_per_thread_stream(fake):
    """One handle stands for a stream of every thread: no order among its calls."""
    assert fake(stream=2) == ("unsplit", None, 2) and not fake.state["taken"]


def test_lora_workspace_never_above_two_partials_of_16_steps():
    """Narrow units keep one partial a workgroup; however finely they are split, no call asks for
    more than two partials a workgroup of ranges of whole rounds of 16 k-steps take."""
    import random

    rng = random.Random(5)
    for _ in range(20000):
        K, M = int(2 ** rng.uniform(9, 18)), 16 * rng.randrange(1, 31 * 16 + 1)
        r = 2 * rng.randrange(1, 60)
        S, KS = -(-M // 256), -(-K // 32)
        most = 256 // S
        rounds = -(-KS // (16 * most))
        parts = -(-KS // (16 * rounds))
        blocks = -(-min(r, 80) // 16)
        assert hilore.hilore_lora_grad_workspace_bytes(K, M, r) <= 2 * S * parts * blocks * 16384, \
            (K, M, r)
