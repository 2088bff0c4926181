"""GPU parity of the general GEMMs at the edges of their block tiles, in every
tile shape, operand alignment and split that the host chooses between, against
the CPU oracle.  Tolerances as in test_gpu_parity (bfloat16 operands): 2e-2 by
Frobenius norm and per row and column."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import lrqat_oracle as O
from test_gpu_parity import rel_fro
from test_gpu_parity_next import Layer, check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_06385_amd import lrqat
    lrqat.load_library()
    return lrqat


CASES = [
    # m, k, T, r, bits, fmt, g, act, asym
    (129, 255, 513, 8, 4, "q8", 0, 0, False),            # odd rows everywhere, one past the 128-row tiles
    (130, 258, 514, 5, 4, "int_packed2", 0, 0, True),    # rows on dwords, a partial K-tile, zero offset
    (131, 320, 520, 32, 6, "q8", 0, 0, False),           # m odd (dX, dW rows), k a whole number of K-tiles
    (192, 323, 576, 16, 3, "q8", 0, 0, False),           # k odd, m aligned
    (256, 1030, 1300, 20, 4, "int_packed2", 0, 0, False),  # dW in ranges of the tokens, unaligned rows
    (264, 512, 2050, 33, 4, "q8", 128, 0, True),         # dW in ranges of the tokens, groups with offsets
    (256, 4096, 2048, 4, 4, "int_packed2", 0, 0, False),
    (128, 11008, 640, 4, 4, "int_packed2", 0, 0, False),
    (4096, 128, 2048, 4, 4, "q8", 0, 0, False),
    (320, 640, 530, 8, 4, "int_packed2", 0, 8, True),    # int8 forward with a zero offset
    (257, 384, 600, 8, 6, "q8", 0, 8, True),             # int8 forward on an int8 grid
    (136, 1000, 520, 8, 4, "int_packed2", 0, 8, False),  # int8 forward, k no multiple of its 128-value K-tile
    (136, 640, 520, 8, 4, "q8", 64, 8, False),           # int8 tokens widened (group-wise scales)
]


@pytest.mark.parametrize("case", CASES, ids=[f"m{s[0]}k{s[1]}T{s[2]}r{s[3]}b{s[4]}g{s[6]}a{s[7]}{'z' if s[8] else ''}" for s in CASES])
def test_tiles(lr, case):
    m, k, T, r, bits, fmt, g, act, asym = case
    c = Layer(lr, m, k, T, r, float(r), bits, fmt, g, act, "bf16", asym=asym, seed=500 + m, b_std=0.02,
              shift=0.01 if asym else 0.0)
    c.check_setup()
    check_layer(lr, c)


def test_nan_stays_in_its_rows(lr):
    """Rows that are not 16-byte aligned are loaded past their end (into the next row) and masked: a NaN at
    the start of a row must not reach the row before it."""
    c = Layer(lr, 140, 201, 560, 8, 8.0, 4, "q8", 0, 0, "bf16", seed=77)
    X, dY = c.d_X.clone(), c.d_dY.clone()
    ref = lr.lrqat_forward(c.spec, c.d_X, c.d_phi, c.d_s, c.d_A, c.d_B)
    base = lr.lrqat_backward(c.spec, c.d_X, c.d_phi, c.d_s, c.d_A, c.d_B, c.d_dY)
    X[50, :8] = float("nan")
    dY[61, :8] = float("inf")
    Y = lr.lrqat_forward(c.spec, X, c.d_phi, c.d_s, c.d_A, c.d_B)
    got = lr.lrqat_backward(c.spec, c.d_X, c.d_phi, c.d_s, c.d_A, c.d_B, dY)
    torch.cuda.synchronize()
    keep = [t for t in range(560) if t != 50]
    assert torch.equal(Y[keep], ref[keep]) and Y[50].isnan().all()
    keep = [t for t in range(560) if t != 61]
    assert torch.equal(got[0][keep], base[0][keep])
    rows = list(range(8, 140))
    assert torch.equal(got[1][rows], base[1][rows])


@pytest.mark.parametrize("m,k,T", [(129, 255, 513), (131, 320, 577), (256, 323, 321)])
def test_bytes_past_a_tensor_stay_out(lr, m, k, T):
    """An odd number of bfloat16 elements ends in the middle of a dword; the vector loads read that
    dword whole, and the two bytes past the tensor (NaNs here) must not enter any sum."""
    c = Layer(lr, m, k, T, 8, 8.0, 4, "q8", 0, 0, "bf16", seed=91)

    def tight(x):
        buf = torch.full((x.numel() + 64,), float("nan"), dtype=x.dtype, device="cuda")
        buf[: x.numel()] = x.flatten()
        return buf[: x.numel()].view(x.shape)

    c.d_X, c.d_dY = tight(c.d_X), tight(c.d_dY)
    check_layer(lr, c)


# Outputs large enough for the larger tiles, with each form of the weight operand.
LARGE = [
    (4096, 192, 2304, 4, 4, "q8", 0, 0, True),
    (4096, 192, 2304, 4, 6, "q8", 0, 0, False),
    (4096, 192, 2304, 4, 7, "q8", 0, 0, True),
    (4096, 256, 2304, 4, 3, "q8", 128, 0, True),
    (4096, 256, 2304, 4, 6, "q8", 128, 0, False),
    (4096, 200, 2304, 4, 4, "int_packed2", 0, 8, False),
    (4096, 200, 2304, 4, 4, "q8", 0, 8, True),
    (4096, 200, 2304, 4, 6, "q8", 0, 8, True),
    (4096, 256, 2304, 4, 4, "int_packed2", 64, 8, True),
    (4096, 128, 2048, 4, 6, "q8", 0, 0, True),
    (4096, 128, 2048, 4, 4, "q8", 64, 0, True),
    (192, 4096, 2304, 4, 4, "q8", 0, 0, True),
    (192, 4096, 2304, 4, 6, "q8", 0, 0, False),
    (192, 4096, 2304, 4, 6, "q8", 128, 0, True),
    (256, 4096, 2048, 4, 6, "q8", 0, 0, True),
    (256, 4096, 2048, 4, 4, "q8", 128, 0, True),
    (128, 11008, 640, 4, 6, "q8", 0, 0, True),
    (128, 10880, 768, 4, 6, "q8", 128, 0, True),
]

# The tiles (and token ranges) that the host chooses for cases of these lists: (GEMM, m, k, T, group, act).
REACHED = {
    (256, 256, 1): [("fwd", 4096, 192, 2304, 0, 0), ("fwd", 4096, 256, 2304, 128, 0), ("fwd", 4096, 200, 2304, 0, 8),
                    ("fwd", 4096, 256, 2304, 64, 8), ("dx", 192, 4096, 2304, 0, 0), ("dx", 192, 4096, 2304, 128, 0),
                    ("dw", 2901, 2903, 66, 0, 0), ("dw", 2902, 2906, 66, 0, 0), ("dw", 2901, 2944, 66, 128, 0)],
    (256, 128, 1): [("fwd", 4096, 128, 2048, 0, 0), ("fwd", 4096, 128, 2048, 64, 0), ("dx", 256, 4096, 2048, 0, 0),
                    ("dx", 128, 10880, 768, 128, 0), ("dw", 2050, 2100, 70, 0, 0), ("dw", 2051, 2101, 130, 0, 0),
                    ("dw", 2056, 2176, 64, 128, 0)],
    (128, 256, 1): [("dx", 128, 11008, 640, 0, 0), ("dx", 256, 4096, 2048, 128, 0)],
    (128, 128, 1): [("fwd", 136, 640, 520, 64, 8), ("fwd", 257, 384, 600, 0, 8), ("fwd", 129, 255, 513, 0, 0),
                    ("dx", 129, 255, 513, 0, 0), ("dw", 129, 255, 513, 0, 0), ("dx", 264, 512, 2050, 128, 0)],
    (128, 128, 2): [("dw", 129, 257, 1030, 0, 0)],
    (128, 128, 4): [("dw", 384, 640, 2050, 128, 0)],
    (128, 128, 16): [("dw", 130, 130, 8192, 0, 0)],
}


@pytest.mark.parametrize("case", LARGE, ids=[f"m{s[0]}k{s[1]}T{s[2]}b{s[4]}g{s[6]}a{s[7]}{'z' if s[8] else ''}" for s in LARGE])
def test_large_tiles(lr, case):
    m, k, T, r, bits, fmt, g, act, asym = case
    c = Layer(lr, m, k, T, r, float(r), bits, fmt, g, act, "bf16", asym=asym, seed=800 + k + bits, b_std=0.02,
              shift=0.01 if asym else 0.0)
    check_layer(lr, c)


DW = [
    # m, k, T, r, bits, fmt, g, asym
    (2050, 2100, 70, 5, 4, "int_packed2", 0, False),     # rows on dwords, past the 256 x 128 tiles in both directions
    (2051, 2101, 130, 33, 4, "q8", 0, False),            # odd rows, ranks past one block of 32
    (2056, 2176, 64, 8, 3, "int_packed2", 128, True),    # groups and offsets, 16-byte rows
    (2901, 2903, 66, 8, 4, "q8", 0, False),              # 256 x 256 tiles with odd rows
    (2902, 2906, 66, 4, 4, "int_packed2", 0, True),      # and rows on dwords, offsets
    (2901, 2944, 66, 4, 4, "q8", 128, False),            # and groups
    (129, 257, 1030, 32, 6, "q8", 0, False),             # two ranges of tokens (8 and 9 K-tiles), odd rows
    (384, 640, 2050, 20, 4, "int_packed2", 128, False),  # four ranges, a last K-tile of two tokens, groups
    (130, 130, 8192, 8, 4, "q8", 0, True),               # 16 ranges, offsets, rows on dwords
]


@pytest.mark.parametrize("case", DW, ids=[f"m{s[0]}k{s[1]}T{s[2]}r{s[3]}b{s[4]}g{s[6]}{'z' if s[7] else ''}" for s in DW])
def test_dw_tiles_and_token_ranges(lr, case):
    m, k, T, r, bits, fmt, g, asym = case
    c = Layer(lr, m, k, T, r, float(r), bits, fmt, g, 0, "bf16", asym=asym, seed=600 + m, b_std=0.02,
              shift=0.01 if asym else 0.0)
    check_layer(lr, c)


@pytest.mark.parametrize("m,k,T,r", [(256, 256, 4096, 32), (500, 701, 1999, 20), (1024, 4096, 1024, 32)])
def test_cancelling_tokens(lr, m, k, T, r):
    """Tokens whose parts of dW nearly cancel: all of them meet in float32 before G is rounded, however the
    tokens are shared out.  dA and dB then carry two bfloat16 roundings a term (G, and B or A), each at most
    2^-9 of it: below 2 * 2^-9 = 3.9e-3 together, 5e-3 with the rest.
    The float32 sums, of parts 64 times the result, add 64 * 2^-24 sqrt(T) < 3e-4."""
    c = Layer(lr, m, k, T, r, float(r), 4, "q8", 0, 0, "bf16", seed=700 + m, b_std=1e-3)
    h = T // 2
    c.d_X[h:2 * h] = c.d_X[:h]
    c.d_dY[h:2 * h] = -(c.d_dY[:h].float() * (1 + 2.0 ** -6)).bfloat16()
    _, dA, dB = lr.lrqat_backward(c.spec, c.d_X, c.d_phi, c.d_s, c.d_A, c.d_B, c.d_dY, want_dx=False)
    torch.cuda.synchronize()
    host = lambda t: t.float().cpu().numpy().astype(np.float64)
    gr = O.backward(c.L, host(c.d_X), c.phi_ref, c.s_ref, c.A, c.B, host(c.d_dY))
    for name, got in (("dA", dA), ("dB", dB)):
        e = rel_fro(got.cpu().numpy(), gr[name])
        assert e < 5e-3, (name, e)
