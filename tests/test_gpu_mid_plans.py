"""GPU parity of the mid kernel's plans: 64-token blocks (two token tiles per
wavefront), and the plans that stand in for the large and prefill kernels,
whose Y is bit-exact with the oracle."""
import pytest

import paper_2606_01556_amd as tq
from test_gpu_parity import full_parity, say
from tq_synth import random_codes_layer

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tq.lib()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("M,K,N,r,group,bf16", [
    (193, 576, 4768, 64, 64, False),    # odd token tiles (half a block past M), a chunk of one block
    (130, 64, 13000, 64, 64, False),    # a single K-group
    (200, 1152, 8000, 16, 128, True),   # 128-wide groups, half a chunk at the end of K
    (161, 512, 10010, 0, 64, False),    # no H: all eight columns residual, ragged N
    (350, 640, 5000, 128, 128, False),  # a 128-rank group in two blocks
    (193, 384, 5000, 0, 128, True),     # the other widths of each rank
    (225, 320, 5000, 16, 64, False),
    (193, 384, 5001, 64, 128, False),
    (193, 320, 5000, 128, 64, True),
])
def test_two_token_tiles(oracle_mod, M, K, N, r, group, bf16):
    """Enough column tiles that 32-token blocks would take a second round over
    the CUs, so the plan of least time has 64-token blocks; Y in the oracle's
    order there, so bit-exact although the kernel is named "mid"."""
    say(f"two token tiles M={M} K={K} N={N} r={r} group={group}")
    assert tq.dual_gemm_block(tq.weight_desc_init(N, K, r, group), M)[0] == 64
    d = random_codes_layer(M, K, N, r, seed=M + N + r)
    g, o = full_parity(oracle_mod, d["X"], d["W_res"], d["L1"], d["L2"], bf16=bf16, group=group)
    assert g["kernel"] == "mid"
    assert (g["Ybits"] == (o["Ybf"] if bf16 else o["Y16"].view("uint16"))).all()


@pytest.mark.parametrize("M,K,N,r,group,kernel,block", [
    (577, 2176, 3430, 128, 128, "large", (32, 128)),   # four column tiles
    # 64-token blocks at every rank and width, an odd number of token tiles
    (1025, 640, 8890, 0, 64, "large", (64, 256)),
    (577, 640, 5250, 0, 128, "large", (64, 256)),
    (961, 640, 8501, 16, 64, "large", (64, 224)),
    (577, 640, 5250, 16, 128, "large", (64, 224)),
    (1025, 640, 7200, 64, 64, "large", (64, 192)),
    (577, 1664, 5250, 64, 128, "large", (64, 192)),
    (577, 1664, 5250, 128, 64, "large", (64, 128)),
    (577, 1664, 3430, 128, 128, "large", (64, 128)),
    (570, 4096, 14300, 128, 64, "prefill", (64, 128)),
])
def test_in_place_of_large_blocks(oracle_mod, M, K, N, r, group, kernel, block):
    """Past 512 tokens (fp8 activation codes) where 128 x 256 blocks fill the
    CUs badly: the mid kernel's blocks run under the other kernel's name, and Y
    stays bit-exact (full_parity demands it under these names)."""
    say(f"in place of {kernel} M={M} K={K} N={N} r={r} group={group}")
    assert tq.dual_gemm_block(tq.weight_desc_init(N, K, r, group), M) == block
    d = random_codes_layer(M, K, N, r, seed=M + N + r)
    g, _ = full_parity(oracle_mod, d["X"], d["W_res"], d["L1"], d["L2"], group=group)
    assert g["kernel"] == kernel


@pytest.mark.parametrize("M,N,r", [(33, 300, 128), (200, 8000, 64)])
@pytest.mark.parametrize("K,group", [(128, 64), (256, 64), (320, 64), (768, 64), (1088, 64), (1408, 64),
                                     (128, 128), (640, 128), (1024, 128), (1152, 128)])
def test_end_of_k(oracle_mod, M, N, r, K, group):
    """The last chunk of K ends with the four groups that hold the last block: one
    block in it, four, five, twelve; 32- and 64-token blocks."""
    say(f"mid end of K M={M} K={K} N={N} r={r} group={group}")
    d = random_codes_layer(M, K, N, r, seed=M + K)
    g, _ = full_parity(oracle_mod, d["X"], d["W_res"], d["L1"], d["L2"], group=group)
    assert g["kernel"] == "mid"


@pytest.mark.parametrize("M,K,N,r,kernel", [(1025, 512, 4100, 16, "large"), (577, 256, 14300, 128, "prefill")])
def test_forced_tiles_leave_other_kernels(M, K, N, r, kernel):
    """mid_tiles of the debug entry applies to the mid kernel: where another kernel
    is named, Y is that kernel's to the bit, not a sum over parts of K."""
    say(f"forced tiles M={M} K={K} N={N} r={r}")
    gen = torch.Generator("cuda").manual_seed(M)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda").half()
    lay = tq.Layer(draw(N, K), draw(K, r), draw(r, N))
    assert tq.dual_gemm_kernel(lay.desc, M) == kernel and tq.dual_gemm_block(lay.desc, M) == (128, 256)
    xc, xs = tq.empty_act(M, K)
    tq.quant_act(draw(M, K), xc, xs)
    y = {}
    for name, tiles in ((kernel, 0), (None, 1), (None, 2), (None, 4)):
        y[tiles] = torch.empty((M, N), dtype=torch.half, device="cuda")
        tq.dual_gemm_debug(lay.desc, lay.packed, xc, xs, M, y[tiles], kernel=name, mid_tiles=tiles)
        assert torch.equal(y[tiles].view(torch.int16), y[0].view(torch.int16)), tiles
