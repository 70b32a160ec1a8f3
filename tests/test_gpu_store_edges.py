"""Where the 32x32 output tiles' stores end: ragged rows and columns, even and odd
N (odd: every second row starts on two bytes only), for each kernel that stores
such tiles.  What lies before and after Y stays as it was."""
import pytest

import paper_2606_01556_amd as tq

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tq.lib()
    yield
    torch.cuda.synchronize()


def store(layer, x, kernel, bf16):
    """Y's bits by the forced kernel, out of a buffer with 64 guard values on
    each side of Y that have to stay."""
    m, n = x.shape[0], layer.desc.n
    xc, xs = tq.empty_act(m, x.shape[1], group=layer.desc.group)
    tq.quant_act(x, xc, xs, layer.desc.group)
    buf = torch.full((64 + m * n + 64,), 0x5a5a, dtype=torch.int16, device="cuda")
    y = buf[64:64 + m * n].view(torch.bfloat16 if bf16 else torch.half).view(m, n)
    tq.dual_gemm_debug(layer.desc, layer.packed, xc, xs, m, y, bf16=bf16, kernel=kernel)
    torch.cuda.synchronize()
    assert (buf[:64] == 0x5a5a).all() and (buf[64 + m * n:] == 0x5a5a).all()
    return y


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("m,k,n,r,group", [
    (33, 128, 34, 8, 64),       # two columns per store, one row and two columns in the last tiles
    (47, 256, 97, 16, 128),     # odd N: one column per store
    (65, 192, 4770, 64, 64),
    (513, 128, 258, 8, 64),     # past 512 tokens: the large and prefill kernels
    (545, 256, 353, 128, 128),
    (634, 256, 1021, 64, 128),
])
def test_stores_end_at_the_tile(m, k, n, r, group, bf16):
    """Nothing around Y is written, and every kernel stores the same value at
    the same place: bit-equal between the two that add in ascending order; a
    mid call equals the decode kernel's on 16-token slices (same codes, exact
    products; the fp32 sums differ in order only) to two output roundings."""
    print(f"store edges m={m} k={k} n={n} r={r} group={group} bf16={bf16}", flush=True)
    gen = torch.Generator("cuda").manual_seed(m + n)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda").half()
    layer = tq.Layer(draw(n, k), draw(k, r), draw(r, n), group=group)
    x = draw(m, k)
    if m > 512:
        y, want = store(layer, x, "large", bf16), store(layer, x, "prefill", bf16)
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))
    else:
        y = store(layer, x, "mid", bf16).float()
        want = torch.cat([store(layer, x[i:i + 16].contiguous(), "decode", bf16).float()
                          for i in range(0, m, 16)])
        # an ulp of the output type, plus K/64 + 2 fp32 roundings of sums no larger
        # than the largest |Y| times the terms that add to it
        tol = want.abs() * 2.0 ** (-7 if bf16 else -10) + want.abs().max() * k * 2.0 ** -24
        assert ((y - want).abs() <= tol).all()


@pytest.mark.parametrize("k,r,group", [(64, 128, 64), (192, 128, 64), (64, 64, 64), (256, 64, 64),
                                       (128, 128, 128), (256, 64, 128)])
def test_prefill_short_k(k, r, group):
    """K loops shorter than the prefill kernel's ring, over a run of three column
    blocks (more token blocks than CUs): the fill repeats the last block, the
    next column block's fill is issued ahead of the epilogue."""
    m, n = 257 * 128 - 5, 600
    print(f"prefill short k={k} r={r} group={group}", flush=True)
    gen = torch.Generator("cuda").manual_seed(k + r)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda").half()
    layer = tq.Layer(draw(n, k), draw(k, r), draw(r, n), group=group)
    x = draw(m, k)
    y, want = store(layer, x, "prefill", False), store(layer, x, "large", False)
    assert torch.equal(y.view(torch.int16), want.view(torch.int16))
