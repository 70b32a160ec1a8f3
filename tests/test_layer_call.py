"""The whole-layer entry (tq_layer) and Layer.__call__: argument checks and
scratch sizes on the CPU, the same bits as the quantizer and the fused layer
called one after the other on the GPU."""
import copy

import numpy as np
import pytest

import paper_2606_01556_amd as tq
from tq_synth import random_codes_layer

torch = pytest.importorskip("torch")
FAKE = 1 << 20     # 16-byte aligned fake device address; never dereferenced


def test_scratch_sizes():
    """0 where the layer is one launch (few tokens, and few values for every
    work-group to quantize), else the binding's own formula."""
    L = tq.lib()
    for n, k, r, g in ((512, 512, 16, 64), (4096, 4096, 64, 64), (4096, 14336, 64, 128), (256, 28672, 128, 64),
                       (128, 65536, 64, 64), (64, 131072, 0, 128)):
        d = tq.weight_desc_init(n, k, r, g)
        for m in (1, 2, 7, 8, 9, 16, 17, 512, 513, 1000):
            got = L.tq_layer_scratch_bytes(d, m)
            one = m <= 16 and min(m, 8) * k <= 32768
            assert got == (0 if one else tq.layer_scratch_bytes(m, k, g)), (k, m)
    assert L.tq_layer_scratch_bytes(d, 0) == 0 and L.tq_layer_scratch_bytes(tq.WeightDesc(), 100) == 0


def test_validation():
    L = tq.lib()
    d = tq.weight_desc_init(128, 4096, 64)
    call = lambda dd=d, p=FAKE, x=FAKE, m=100, y=FAKE, t=0, s=FAKE: L.tq_layer(dd, p, x, m, y, t, s, None)
    assert call(dd=None) == 1 and call(p=None) == 1 and call(x=None) == 1 and call(y=None) == 1
    assert call(s=None) == 1                        # two launches need scratch
    assert call(dd=tq.WeightDesc()) == 7
    assert call(m=-1) == 2 and call(m=65535 * 32 + 1) == 2
    assert call(t=5) == 5 and call(t=5, m=1) == 5
    assert call(x=FAKE + 8) == 6 and call(s=FAKE + 8) == 6 and call(y=FAKE + 2, m=1) == 6
    assert call(m=0) == 0


class FakeGpuTensor(torch.Tensor):
    """A host tensor that passes for a GPU one; the stand-in library below takes
    its address and follows none."""
    is_cuda = property(lambda self: True)


class FakeLib:
    """Records the pointers of tq_layer; the rest is the library's own."""

    def __init__(self):
        self.calls, self.real = [], tq.lib()

    def tq_layer(self, *args):
        self.calls.append(args)
        return 0

    def __getattr__(self, name):
        return getattr(self.real, name)


@pytest.fixture
def fake(monkeypatch):
    """(library, layer, x) for Layer.__call__ without a GPU."""
    fake = FakeLib()
    monkeypatch.setattr(tq, "lib", lambda: fake)
    monkeypatch.setattr(tq, "_current_stream", lambda: 0)
    gpu = lambda *s, dtype=torch.float16: torch.empty(s, dtype=dtype).as_subclass(FakeGpuTensor)
    lay = tq.Layer.__new__(tq.Layer)
    lay.desc = tq.weight_desc_init(96, 512, 16)
    lay.packed = gpu(lay.desc.packed_bytes, dtype=torch.uint8)
    lay.n, lay.k, lay.rank = 96, 512, 16
    return fake, lay, gpu(3, 512)


def test_packed_and_desc_are_checked(fake):
    """What the library would read out of bounds is refused before the call: packed
    weights on the host, too short or strided, and a descriptor of other sizes; a
    raw device address is taken as it is."""
    L, lay, x = fake
    packed, desc = lay.packed, lay.desc
    lay(x)
    assert len(L.calls) == 1 and L.calls[0][1] == packed.data_ptr()
    for bad in (torch.empty(packed.numel(), dtype=torch.uint8), packed[:-1],
                torch.empty(2 * packed.numel(), dtype=torch.uint8).as_subclass(FakeGpuTensor)[::2], None):
        lay.packed = bad
        with pytest.raises(ValueError):
            lay(x)
    lay.packed = packed
    for n, k in ((128, 512), (96, 576)):
        lay.desc = tq.weight_desc_init(n, k, 0)
        with pytest.raises(ValueError):
            lay(x)
    lay.desc = desc
    assert len(L.calls) == 1
    lay.packed = FAKE
    lay(x)
    assert L.calls[1][1] == FAKE


def test_result_is_a_plain_tensor(fake):
    """Also for activations of a tensor subclass."""
    L, lay, x = fake
    assert type(x) is FakeGpuTensor and type(lay(x)) is torch.Tensor
    y = lay(x, bf16=True)
    assert type(y) is torch.Tensor and y.dtype == torch.bfloat16 and y.shape == (3, 96)


def test_only_the_saved_attributes(fake):
    """A layer needs no more than desc, packed, n, k and rank, which a program may
    have saved or set by itself; scratch where the size asks for it."""
    L, lay, x = fake
    lay(x)
    assert L.calls[-1][6] is None
    lay(torch.empty((17, 512), dtype=torch.float16).as_subclass(FakeGpuTensor))
    assert L.calls[-1][6] is not None


@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n,r,group,bf16", [
    (1, 4096, 300, 64, 64, False), (8, 4096, 300, 64, 64, True), (8, 4160, 300, 64, 64, False),
    (16, 512, 96, 16, 128, False), (16, 4160, 96, 16, 64, True), (17, 256, 100, 0, 64, False),
    (513, 256, 100, 32, 64, False), (1, 32768, 64, 16, 64, False), (1, 40960, 64, 16, 64, False),
])
def test_layer_call(m, k, n, r, group, bf16):
    """Either side of the one-launch rule, of the 4-bit / fp8 code formats, and
    on another stream than the current one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case]", m, k, n, r, group, bf16, flush=True)
    d = random_codes_layer(m, k, n, r, seed=m + k)
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    lay = tq.Layer(dev(d["W_res"]), dev(d["L1"]), dev(d["L2"]), group=group)
    x = dev(d["X"])
    xc, xs = tq.empty_act(m, k, group=group)
    tq.quant_act(x, xc, xs, group)
    ref = torch.empty((m, n), dtype=torch.bfloat16 if bf16 else torch.float16, device="cuda")
    tq.dual_gemm(lay.desc, lay.packed, xc, xs, m, ref, bf16)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for layer, stream in ((lay, None), (lay, side), (copy.deepcopy(lay), None)):
        y = layer(x, bf16, stream=stream)
        torch.cuda.synchronize()
        assert y.dtype == ref.dtype and torch.equal(y.view(torch.int16), ref.view(torch.int16))
    if m == 1:      # needs no scratch at any K
        y.fill_(-1.0)
        assert 0 == tq.lib().tq_layer(lay.desc, lay.packed.data_ptr(), x.data_ptr(), m, y.data_ptr(), 1 if bf16 else 0, None,
                                      torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16))


def stream_of(t):
    """The hipStream_t whose memory the allocator took t's storage from."""
    for seg in torch.cuda.memory_snapshot():
        if seg["address"] <= t.data_ptr() < seg["address"] + seg["total_size"]:
            return seg["stream"]


@pytest.mark.gpu
def test_other_stream():
    """A call on another stream than the current one works in that stream's memory
    -- given as a torch stream, its handle, the default stream and 0 -- so
    nothing pending on the current stream, where a block of the same size was
    just freed, can touch its codes or its result."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator("cuda").manual_seed(3)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda").half()
    m, k, n = 600, 1024, 1000
    lay = tq.Layer(draw(n, k), draw(k, 32), draw(32, n))
    x = draw(m, k)
    want = lay(x)
    torch.cuda.synchronize()
    side, here = torch.cuda.Stream(), torch.cuda.Stream()
    default = torch.cuda.default_stream()
    busy = torch.randn(2048, 2048, device="cuda")
    for current, given in ((default, side), (default, side.cuda_stream), (here, side), (here, default), (here, 0)):
        print("[case] current", current, "given", given, flush=True)
        with torch.cuda.stream(current):
            handle = given if isinstance(given, int) else given.cuda_stream
            old = [torch.empty(b, dtype=torch.uint8, device="cuda")
                   for b in (tq.layer_scratch_bytes(m, k), m * n * 2)]
            for _ in range(20):
                busy = busy @ busy * 1e-3
            for t in old:
                t.fill_(0x77)          # behind the products: pending when freed
            del old, t
            y = lay(x, stream=given)
            assert stream_of(y) == handle
            torch.cuda.ExternalStream(handle).synchronize() if handle else default.synchronize()
            assert torch.equal(y.view(torch.int16), want.view(torch.int16))
        torch.cuda.synchronize()
    assert stream_of(lay(x, stream=default)) == default.cuda_stream      # the current one, by its name
