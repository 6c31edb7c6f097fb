"""The bulk encode on the matrix cores stores codes of sums that it has rounded, where a bound says that no comparison
can differ from that of the exact sums.  Here: the bound on the instruction's own rounding, and ranges long enough
for that kernel whose coefficients lie within rounding of a threshold, at both ends of the range, and on zero."""

import ctypes
import os

import numpy as np
import pytest
import torch

import synth_inputs as synth

pytestmark = pytest.mark.gpu

# vectors from which the launcher takes the matrix cores, and the ones whose index m has H_{2^m} in H_d
LONG = {64: 1, 96: 192 << 10, 160: 384 << 10, 192: 64 << 10, 256: 192 << 10}
BLOCK = {64: 1, 96: 12, 160: 20, 192: 12, 256: 1}


def bits_of(x):
    """bf16 bits of numbers that bf16 holds."""
    b = (np.ascontiguousarray(x, dtype=np.float32).view(np.uint32) >> np.uint32(16)).astype(np.uint16)
    assert np.array_equal(synth.bf16_bits_to_f32(b), x)
    return b


def rounded(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).bfloat16().float().numpy()


def check(oracle, rows, d, thr, bits):
    """`rows` (bf16 bits [n][d]), repeated until the range is long enough (and ends in mid-step): the oracle's codes."""
    import paper_2510_18413_amd as A
    n = rows.shape[0]
    copies = (LONG[d] + 21 + n - 1) // n
    K = torch.from_numpy(rows.view(np.int16)).view(torch.bfloat16).cuda().repeat(copies, 1)[None].contiguous()
    cfg = A.Config.make(1, 1, n * copies, thr_k=thr, head_dim=d, code_bits=0 if bits == 2 else bits)
    codes = torch.full((1, n * copies, cfg.code_row_bytes), 0xEE, dtype=torch.uint8, device="cuda")
    A.adamas_encode_keys(cfg, K, codes, 0, n * copies)
    with oracle.head_dim(d):
        ref = torch.from_numpy(oracle.encode_bits(rows, thr, bits)[1]).cuda()
    wrong = (codes.view(copies, n, -1) != ref).any(-1)
    assert not bool(wrong.any()), wrong.nonzero()[:4].tolist()


@pytest.mark.parametrize("form", ["spread", "truncated", "cancelling"])
def test_rounding_of_the_matrix_instruction(form):
    """With u = 2^-24: at most 12 u sum |x| by the model that the certificate follows (it allows for 32 u)."""
    path = os.path.join(os.path.dirname(__file__), "libmatrix_sums.so")
    if not os.path.exists(path):
        import __graft_entry__
        __graft_entry__.build_matrix_sums()
    lib = ctypes.CDLL(path)
    lib.matrix_sums.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_void_p]
    gen = torch.Generator(device="cuda").manual_seed(9)
    worst, tiles = 0.0, 4096
    for spread in (0, 3, 9, 14, 28):
        signs = torch.where(torch.rand(tiles, 16, 32, generator=gen, device="cuda") < 0.5, -1.0, 1.0)
        x = 1 + torch.rand(tiles, 32, 16, generator=gen, device="cuda")
        if form == "spread":
            x *= torch.exp2(torch.randint(-spread, 1, x.shape, generator=gen, device="cuda").float())
            x *= torch.where(torch.rand(x.shape, generator=gen, device="cuda") < 0.5, -1.0, 1.0)
        else:
            # one large element per eight, the others just above and below what is kept beside it
            small = torch.exp2(-torch.randint(14, 20 + spread // 2, x.shape, generator=gen, device="cuda").float())
            at = torch.randint(0, 8, (tiles, 4, 1, 16), generator=gen, device="cuda")
            first = torch.zeros(tiles, 4, 8, 16, device="cuda").scatter_(2, at, 1.0).view_as(x).bool()
            x = torch.where(first, x.round(), x * small)
            if form == "cancelling":       # the large ones in pairs of opposite signs under the signs of row 0
                flip = torch.tensor([1.0, -1.0, 1.0, -1.0], device="cuda").repeat_interleave(8)[:, None]
                x = torch.where(first, flip * signs[:, 0, :, None], x)
            else:
                signs[:, 0] = 1
        B = x.bfloat16().contiguous()
        A = signs.bfloat16().contiguous()
        D = torch.full((tiles, 16, 16), float("nan"), device="cuda")
        torch.cuda.synchronize()
        assert lib.matrix_sums(A.data_ptr(), B.data_ptr(), D.data_ptr(), tiles, torch.cuda.current_stream().cuda_stream) == 0
        exact = torch.bmm(A.double(), B.double())
        err = (D.double() - exact).abs() / (2.0 ** -24 * B.double().abs().sum(1, keepdim=True))
        worst = max(worst, float(err.max()))
    print("worst error / (u sum |x|): %.3f" % worst)
    assert worst <= 12.0


def hadamard_variants(x, d):
    """x times the rows of H_{2^n} (d = 2^n m): the same coefficients in other places, summed in another order."""
    m = BLOCK[d]
    r = np.arange(d // m)
    par = np.array([[bin(a & b).count("1") & 1 for b in r] for a in r])
    return np.repeat(1.0 - 2.0 * par, m, axis=1).astype(np.float32) * x


@pytest.mark.parametrize("d", [64, 96, 160, 192, 256])
@pytest.mark.parametrize("kind", ["one bit", "symmetric", "unsymmetric"])
def test_long_ranges_within_rounding_of_a_threshold(oracle, d, kind):
    rng = np.random.default_rng(31 * d + len(kind))
    bits, above, below = (1 if kind == "one bit" else 2), 0, 0
    for trial in range(6):
        spread = (0, 10, 10, 14, 18, 20)[trial]
        x = rng.standard_normal((384, d), dtype=np.float32) * np.exp2(-rng.integers(0, spread + 1, size=(384, d))).astype(np.float32)
        x[0:32:3, d // 2:] = x[0:32:3, :d // 2]          # coefficients that are zero
        x[1:32:3] = 0
        x[2:32:3] = x[2:32:3, :1]
        x = rounded(np.where(np.abs(x) < 2.0 ** -28, 0, x))
        own = [hadamard_variants(x[100 + i], d) for i in range(3)]
        with oracle.head_dim(d):
            picks = [float(oracle.hadamard_transform(x[100 + i].astype(np.float64))[rng.integers(d)]) for i in range(3)]
        tau = lambda v: float(np.float32(v / np.sqrt(float(d))))
        rows = bits_of(np.concatenate([x] + own))
        if kind == "symmetric":
            picks = [abs(p) for p in picks if tau(p) != 0]
        above += sum(p > tau(p) * np.sqrt(float(d)) for p in picks)
        below += sum(p < tau(p) * np.sqrt(float(d)) for p in picks)
        if kind == "one bit":
            forms = [(tau(p),) for p in picks]
        elif kind == "symmetric":
            forms = [(-tau(p), 0.0, tau(p)) for p in picks]
        else:
            forms = [tuple(sorted(tau(p) for p in picks))]
        for thr in forms:
            if len(set(thr)) == len(thr):
                check(oracle, rows, d, thr, bits)
    assert above > 0 and below > 0


@pytest.mark.parametrize("d", [64, 96, 160, 192, 256])
@pytest.mark.parametrize("bits,thr", [(1, (0.13,)), (2, (-1.0, 0.0, 1.0)), (2, (-0.7, 0.13, 0.9))])
def test_long_ranges_of_extreme_magnitudes(oracle, d, bits, thr):
    """Sums near the ends of the fp32 range, below what is certified and above it, and elements spread over 2^28."""
    rng = np.random.default_rng(7 * d + bits)
    x = rounded(rng.standard_normal((512, d), dtype=np.float32))
    x[np.abs(x) < 2.0 ** -7] = 0
    for scale in (2.0 ** 116, 2.0 ** 92, 2.0 ** -100, 2.0 ** -106, 2.0 ** -118):
        check(oracle, bits_of(x * np.float32(scale)), d, tuple(float(np.float32(t * scale)) for t in thr), bits)
    wide = x * np.exp2(rng.integers(-17, 12, size=x.shape)).astype(np.float32)
    check(oracle, bits_of(wide), d, thr, bits)


@pytest.mark.parametrize("d", [64, 96, 160, 192, 256])
@pytest.mark.parametrize("bits,thr", [(1, (0.0,)), (2, (-1e-39, 0.0, 1e-39)), (2, (-1.0, 0.0, 1.0)), (2, (-1e-39, 2e-39, 1.0))])
def test_long_ranges_of_subnormal_elements(oracle, d, bits, thr):
    """Rows of subnormal numbers only, of zeros of either sign, and rows whose subnormal elements decide a code."""
    rng = np.random.default_rng(3 * d + bits)
    rows = (rng.integers(0, 128, size=(512, d)) | rng.integers(0, 2, size=(512, d)) << 15).astype(np.uint16)
    rows[0::8] &= 0x8000
    rows[1::8] = 0
    rows[2::8, 5] = bits_of(np.float32([2.0 ** -118]))
    rows[3::8, 1:] &= 0x8000
    check(oracle, rows, d, thr, bits)
