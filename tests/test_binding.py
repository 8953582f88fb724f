"""The binding's host logic, on the CPU: stand-ins for GPU tensors and streams,
and for the C calls (recorded, not made)."""
import contextlib
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2504_17577_amd import tileattn as ta  # noqa: E402

BF16, F32 = torch.bfloat16, torch.float32


class FakeTensor:
    """What the binding reads of a contiguous GPU tensor."""
    is_cuda, device = True, "cuda:0"

    def __init__(self, shape, dtype, stream=None):
        self.shape = (shape,) if isinstance(shape, int) else tuple(shape)
        self.dtype, self.stream = dtype, stream

    def dim(self):
        return len(self.shape)

    def is_contiguous(self):
        return True

    def get_device(self):
        return 0

    def data_ptr(self):
        return 0x10000000

    def numel(self):
        n = 1
        for s in self.shape:
            n *= s
        return n

    def record_stream(self, stream):
        pass

    def new_empty(self, shape, dtype):
        return torch.empty(shape, dtype=dtype, device=self.device)


class FakeStream:
    cuda_stream = 0x5000


class FakeLib:
    """The library's host helpers, with every launching entry point recorded."""
    LAUNCHES = ("attn_fwd", "attn_fwd_bf16out", "attn_fwd_split", "mla_decode", "gemm_bf16",
                "gemm_bf16_split", "gemv_bf16_split", "ssd_chunk_state", "ssd_state_passing",
                "ssd_bmm_chunk", "ssd_chunk_scan", "ssd_forward")

    def __init__(self, real):
        self.real, self.calls = real, []

    def __getattr__(self, name):
        if name not in self.LAUNCHES:
            return getattr(self.real, name)
        return lambda *args: self.calls.append((name, args)) or 0


@pytest.fixture
def fake(monkeypatch):
    """lib: the recorded C calls; made: the tensors allocated by the binding,
    each with the stream that was current for it."""
    real, current, made = ta.lib(), [None], []

    @contextlib.contextmanager
    def on(stream):
        before, current[0] = current[0], stream
        yield
        current[0] = before

    def empty(shape, dtype=None, device=None):
        made.append(FakeTensor(shape, dtype, current[0]))
        return made[-1]

    lib = FakeLib(real)
    lib.made = made
    monkeypatch.setattr(ta, "_lib", lib)
    monkeypatch.setattr(ta, "_one_device", lambda *t: contextlib.nullcontext())
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 0, raising=False)
    return lib


def t(*shape, dtype=BF16):
    return FakeTensor(shape, dtype)


def ssd_args(B, L, H, G):
    return (t(B, L, H, 64), t(B, L, H, dtype=F32), t(H, dtype=F32), t(B, L, G, 128), t(B, L, G, 128))


CALLS = {
    # the call, and the tensors it allocates for itself (not outputs)
    "gemm": (lambda s: ta.gemm_bf16(t(384, 8256), t(8256, 4224), out=t(384, 4224, dtype=F32), stream=s), 1),
    "gemv": (lambda s: ta.gemv_bf16_split(t(1, 9216), t(9216, 9216), out=t(1, 9216, dtype=F32), stream=s), 1),
    "attn": (lambda s: ta.attn_fwd_split(t(1, 8, 1, 128), t(1, 8, 8192, 128), t(1, 8, 8192, 128),
                                         out=t(1, 8, 1, 128, dtype=F32), lse=t(1, 8, 1, dtype=F32),
                                         stream=s), 1),
    "mla": (lambda s: ta.mla_decode(t(1, 128, 512), t(1, 128, 64), t(1, 4096, 1, 512), t(1, 4096, 1, 64),
                                    out=t(1, 128, 512, dtype=F32), lse=t(1, 128, dtype=F32), stream=s), 1),
    "ssd": (lambda s: ta.ssd_forward(*ssd_args(1, 1000, 64, 1), stream=s), 1),
    "ssd_chained": (lambda s: ta.ssd_forward(*ssd_args(1, 300, (1 << 17) + 1, 1), stream=s), 3),
}


@pytest.mark.parametrize("name", CALLS)
@pytest.mark.parametrize("side", [True, False], ids=["side", "current"])
def test_scratch_is_allocated_on_the_launch_stream(fake, name, side):
    """Memory that a call takes for itself comes from the pool of the stream it
    launches on; outputs come from the current stream's."""
    call, n = CALLS[name]
    s = FakeStream() if side else None
    call(s)
    assert fake.calls, "nothing was launched"
    handle = s.cuda_stream if side else 0
    assert all(args[-1] == handle for _, args in fake.calls)
    assert len([x for x in fake.made if x.dtype == torch.uint8]) == (1 if n == 1 else 0)
    outputs = {"ssd": 2, "ssd_chained": 2}.get(name, 0)
    assert [x.stream for x in fake.made].count(s) == (n if side else n + outputs)
    assert len(fake.made) == n + outputs


def test_gemm_without_memory_for_the_split(fake, monkeypatch):
    """gemm_bf16(a, b, out=c) needs no memory of its own: where the workspace
    of the count it chooses cannot be had, it runs unsplit.  A count that the
    caller chose raises."""
    def full(*args):
        raise torch.OutOfMemoryError("full")

    monkeypatch.setattr(ta, "_scratch", full)
    args = t(384, 8256), t(8256, 4224), t(384, 4224, dtype=F32)
    assert ta.gemm_bf16(*args) is args[2]
    assert [name for name, _ in fake.calls] == ["gemm_bf16"]
    with pytest.raises(torch.OutOfMemoryError):
        ta.gemm_bf16(*args, num_splits=5)


def test_ssd_calls_take_a_false_stream_as_the_current_one(fake):
    """stream=0 means the current stream to the SSD functions."""
    x, dt, A, Bm, Cm = ssd_args(1, 300, 4, 2)
    st = t(1, 2, 4, 64, 128, dtype=F32)
    ta.ssd_chunk_state(x, Bm, dt, A, stream=0)
    ta.ssd_state_passing(st, dt, A, prev=st, stream=0)
    ta.ssd_bmm_chunk(Cm, Bm, stream=0)
    ta.ssd_chunk_scan(x, Cm, t(1, 2, 2, 256, 256, dtype=F32), dt, A, st, stream=0)
    ta.ssd_forward(x, dt, A, Bm, Cm, stream=0)
    assert [args[-1] for _, args in fake.calls] == [0] * 5
    assert all(m.stream is None for m in fake.made)


def test_module_without_torch():
    """The host helpers and the *_raw calls take integers only: the module
    imports and serves them where torch is not installed."""
    code = ("import sys; sys.modules['torch'] = None\n"
            "from paper_2504_17577_amd import tileattn as ta\n"
            "assert ta.ta_split_workspace_bytes(2, 3, 100, 128, 4) == 4 * 2 * 3 * 100 * 129 * 4\n"
            "assert ta.gemm_bf16_raw(0, 0, 0, False, 128, 128, 64, None) == 1\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
