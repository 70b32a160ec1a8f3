"""GPU parity of the decode kernel's wide work-groups (six, twelve and sixteen
column tiles, four or eight wavefronts per pair of K blocks), of the ways a pair's
tiles are shared out, and of its two token blocks."""
import numpy as np
import pytest

import paper_2606_01556_amd as tq
from test_gpu_parity import full_parity, run_gpu, say
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


@pytest.mark.parametrize("M,K,N,r,group", [
    (1, 192, 33000, 128, 64),      # one token, an odd number of K blocks
    (2, 1280, 32800, 16, 128),     # one rank tile, formed by all four wavefronts of a pair
    (5, 640, 32784, 32, 64),       # two rank tiles, each formed twice; a ragged last tile
    (9, 1088, 16500, 64, 64),      # a second token block of one token
    (16, 512, 16400, 128, 128),
    (12, 320, 20000, 0, 64),
    (16, 640, 24576, 8, 64),       # the last N of twelve tiles, and the first of sixteen
    (9, 384, 24577, 128, 64),
    (16, 1280, 24600, 0, 128),
    (12, 64, 24600, 64, 64),
    (5, 192, 49100, 128, 64),      # one token block of twelve tiles
    # one and two tokens: six tiles from K = 2048 on, an odd number of K blocks
    (1, 2048, 16400, 128, 64),
    (2, 2368, 20001, 32, 64),
    (2, 2048, 24576, 16, 128),
    (1, 2112, 24560, 0, 64),
])
def test_wide_work_groups(oracle_mod, M, K, N, r, group):
    """More column tiles (times token blocks) than eight per CU: codes and fp16
    activations in, the same bits out of both, H bit-exact."""
    say(f"decode wide M={M} K={K} N={N} r={r} group={group}")
    d = random_codes_layer(M, K, N, r, seed=M + N + r)
    args = (d["X"], d["W_res"], d["L1"], d["L2"])
    g, _ = full_parity(oracle_mod, *args, group=group)
    assert g["kernel"] == "decode"
    g2 = run_gpu(*args, debug=False, fused_quant=True, group=group)
    np.testing.assert_array_equal(g["Ybits"], g2["Ybits"])


@pytest.mark.parametrize("M,K,N,r,group", [
    # one, two and four wavefronts per pair of K blocks: r = 128, one column tile
    (1, 4096, 300, 128, 128),
    (1, 2560, 300, 128, 64),
    (1, 512, 300, 128, 64),
    # K one pair more than a chunk of four pairs, and an odd number of blocks
    (1, 640, 9000, 64, 128),
    (2, 448, 17000, 32, 64),
    (2, 2048, 9000, 16, 64),
    # up to eight tokens: fewer rank tiles than wavefronts of a pair, and as many
    (5, 320, 9000, 16, 64),
    (7, 1152, 300, 64, 128),
    # two token blocks, eight wavefronts per pair: a single K block, whole and
    # broken chunks of two pairs
    (12, 64, 25000, 64, 64),
    (16, 1280, 24600, 0, 128),
    (9, 384, 24800, 128, 64),
    # either side of the K from which LDS holds one buffer of H products, not two
    (1, 103168, 32, 128, 64), (1, 103232, 32, 128, 64), (2, 53568, 32, 128, 64),
    (8, 21120, 32, 128, 64), (8, 21184, 32, 128, 64),
])
def test_wavefronts_per_pair(oracle_mod, M, K, N, r, group):
    """Short and long K at each way a pair's tiles are shared out: H bit-exact,
    the same bits out of the codes and the fp16 activations."""
    say(f"decode split M={M} K={K} N={N} r={r} group={group}")
    d = random_codes_layer(M, K, N, r, seed=M + N + r)
    args = (d["X"], d["W_res"], d["L1"], d["L2"])
    g, _ = full_parity(oracle_mod, *args, group=group)
    assert g["kernel"] == "decode"
    g2 = run_gpu(*args, debug=False, fused_quant=True, group=group)
    np.testing.assert_array_equal(g["Ybits"], g2["Ybits"])


@pytest.mark.parametrize("M,K,N,r", [(9, 192, 100, 64), (11, 320, 8200, 16), (15, 128, 300, 0)])
def test_odd_token_blocks(oracle_mod, M, K, N, r):
    """9 to 15 tokens, an odd number: the first token block has one more than the
    second; H of both blocks bit-exact."""
    say(f"decode token blocks M={M} K={K} N={N} r={r}")
    d = random_codes_layer(M, K, N, r, seed=M + N + r)
    args = (d["X"], d["W_res"], d["L1"], d["L2"])
    g, _ = full_parity(oracle_mod, *args)
    assert g["kernel"] == "decode"
    g2 = run_gpu(*args, debug=False, fused_quant=True)
    np.testing.assert_array_equal(g["Ybits"], g2["Ybits"])
