"""GPU parity of the few-token forward (weights streamed, K split over a
block's waves), at the edges of its token groups (16, 32, 64) and past them, with partial row groups, partial K chunks and rows at every alignment,
against the CPU oracle.  Tolerances as in test_gpu_parity: bfloat16 outputs and
bfloat16 weight operands, 2e-2 by Frobenius norm and per line."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import lrqat_oracle as O
from test_gpu_parity import TOL, assert_close, errors, from_dev
from test_gpu_parity_next import Layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_06385_amd import lrqat
    lrqat.load_library()
    return lrqat


CASES = [
    # m, k, T, bits, fmt, g, act, asym
    (64, 128, 1, 4, "int_packed2", 0, 0, False),       # one chunk, one wave
    (1000, 4096, 16, 4, "int_packed2", 0, 0, False),   # rows past m in the last group
    (131, 1158, 17, 4, "int_packed2", 0, 0, True),     # odd m, rows not on dwords, partial chunk, zero offset
    (96, 2728, 33, 3, "q8", 0, 0, False),              # dword-aligned rows, k no multiple of 32
    (144, 1023, 5, 4, "q8", 0, 0, False),              # odd k (training forward only)
    (80, 768, 65, 4, "q8", 128, 0, True),              # group-wise scales with zero offsets
    (80, 288, 128, 6, "q8", 32, 0, True),              # int8 grid, groups of one 32-column chunk
    (72, 520, 31, 7, "q8", 0, 0, False),               # int8 grid, per channel
    (640, 1030, 3, 4, "int_packed2", 0, 8, True),      # int8 tokens, int8 MFMA, zero offset
    (160, 4096, 128, 4, "int_packed2", 0, 8, False),   # int8 tokens, two blocks of tokens
    (200, 640, 511, 4, "q8", 0, 0, False),             # the most tokens, rows past m
    (8200, 256, 20, 4, "int_packed2", 0, 0, False),    # two row groups with two token groups
    (96, 640, 64, 6, "q8", 0, 8, True),                # int8 tokens, int8 grid
    (96, 640, 40, 4, "q8", 64, 8, True),               # int8 tokens, group-wise scales (widened to bfloat16)
]


@pytest.mark.parametrize("case", CASES, ids=[f"m{s[0]}k{s[1]}T{s[2]}b{s[3]}g{s[5]}a{s[6]}{'z' if s[7] else ''}" for s in CASES])
def test_few_tokens(lr, case):
    m, k, T, bits, fmt, g, act, asym = case
    c = Layer(lr, m, k, T, 8, 8.0, bits, fmt, g, act, "bf16", asym=asym, seed=220 + m, b_std=0.05, shift=0.01 if asym else 0.0)
    q_ref, _, near, _ = O.grid_from_inputs(c.phi_ref, c.A, c.B, 8.0, 8, bits, fmt)
    Xh = O.layer_input(c.Xv, act)
    W = O.weight_hat(q_ref, c.s_ref, g, c.z_ref)
    Yr, mag = Xh @ W.T, np.abs(Xh) @ np.abs(W).T
    Y = lr.lrqat_forward(c.spec, c.d_X, c.d_phi, c.d_s, c.d_A, c.d_B, z=c.d_z)
    torch.cuda.synchronize()
    assert_close({"Y": errors(from_dev(Y), Yr, mag, TOL["bf16"])}, TOL["bf16"])
    if bits <= 4 and k % 2 == 0:
        # the merged weights give the training forward's bits
        Wz = lr.lrqat_merge_to_int4(c.spec, c.d_phi, c.d_A, c.d_B)
        Yi = lr.lrqat_infer_forward(c.spec, c.d_X, Wz, c.d_s, z=c.d_z)
        torch.cuda.synchronize()
        assert torch.equal(Y.view(torch.int16), Yi.view(torch.int16))


def test_int8_sum_is_exact(lr):
    """Int8 tokens with per-channel scales: the sum of integer products is exact in int32, so Y is
    fl_bf16(fl32(fl32(N s) s_x)) of the integer N = sum n (q - z) (|N| < 2^24 here)."""
    c = Layer(lr, 64, 2048, 48, 8, 8.0, 4, "int_packed2", 0, 8, "bf16", asym=True, seed=311, b_std=0.05, shift=0.01)
    q, _, _, _ = O.grid_from_inputs(c.phi_ref, c.A, c.B, 8.0, 8, 4, "int_packed2")
    _, n, sx = O.act_quant(c.Xv)
    N = n @ (q - np.asarray(c.z_ref)[:, None]).T
    assert np.abs(N).max() < 2 ** 24
    ref = (N.astype(np.float32) * c.s_ref[None, :].astype(np.float32)).astype(np.float32) * sx[:, None].astype(np.float32)
    Y = lr.lrqat_forward(c.spec, c.d_X, c.d_phi, c.d_s, c.d_A, c.d_B, z=c.d_z)
    torch.cuda.synchronize()
    assert torch.equal(Y.cpu(), torch.from_numpy(ref.astype(np.float32)).to(torch.bfloat16))


@pytest.mark.parametrize("k", [40, 1002, 2048, 2056, 8200, 16384, 16408])
def test_token_codes_at_every_row_length(lr, k):
    """Row lengths on both sides of what the token quantisation holds in registers (2048, 4096, 8192 and 16384
    values) and one that is no whole number of 16-byte vectors: the codes are exact, so Y is too, as above
    (|N| <= 127 * 7 * k < 2^24)."""
    c = Layer(lr, 32, k, 5, 4, 4.0, 4, "int_packed2", 0, 8, "bf16", seed=401, b_std=0.02)
    X = c.Xv.copy()
    X[1] = 0.0                  # a token of zeros
    X[2, : k - 1] = 0.0         # its only value, and the maximum, in the last place
    X[3, 0] = 64.0              # and in the first
    d_X = torch.from_numpy(X.astype(np.float32)).to(torch.bfloat16).cuda()
    X = d_X.float().cpu().numpy().astype(np.float64)
    q, _, _, _ = O.grid_from_inputs(c.phi_ref, c.A, c.B, 4.0, 4, 4, "int_packed2")
    _, n, sx = O.act_quant(X)
    N = (n @ q.T).astype(np.float32)
    ref = (N * c.s_ref[None, :].astype(np.float32)).astype(np.float32) * sx[:, None].astype(np.float32)
    Y = lr.lrqat_forward(c.spec, d_X, c.d_phi, c.d_s, c.d_A, c.d_B)
    torch.cuda.synchronize()
    assert torch.equal(Y.cpu(), torch.from_numpy(ref.astype(np.float32)).to(torch.bfloat16))
