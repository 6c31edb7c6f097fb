"""A threshold of -0 is 0 in every encode: rows of zeros of either sign and coefficients that cancel."""

import numpy as np
import pytest
import torch

import synth_inputs as synth

pytestmark = pytest.mark.gpu

# vectors from which the bulk encode takes the matrix cores
LONG = {64: 1, 96: 192 << 10, 160: 384 << 10, 192: 64 << 10, 256: 192 << 10}


def bits_of(x):
    """bf16 bits of numbers that bf16 holds."""
    b = (np.ascontiguousarray(x, dtype=np.float32).view(np.uint32) >> np.uint32(16)).astype(np.uint16)
    assert np.array_equal(synth.bf16_bits_to_f32(b), x)
    return b


def rounded(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).bfloat16().float().numpy()


@pytest.mark.parametrize("d", [64, 96, 128, 160, 192, 256])
@pytest.mark.parametrize("bits,thr", [(1, (-0.0,)), (2, (-0.8, -0.0, 1.0)), (2, (-1.0, -0.0, 1.0)), (3, (-3.0, -2.0, -1.0, -0.0, 1.0, 2.0, 3.0))])
@pytest.mark.parametrize("hadamard", [True, False])
def test_a_threshold_of_negative_zero_is_zero(oracle, d, bits, thr, hadamard):
    import paper_2510_18413_amd as A
    rng = np.random.default_rng(d)
    for n in [50] + ([LONG[d] + 5] if d in LONG and bits <= 2 and hadamard else []):
        x = rounded(rng.standard_normal((n, d), dtype=np.float32))
        x[0::3] = 0
        x[1::9] = -0.0
        x[2::9, ::2] = 0
        cfg = A.Config.make(1, 1, n, thr_k=thr, head_dim=d, code_bits=0 if bits == 2 else bits,
                            variant=0 if hadamard else A.VARIANT_NO_HADAMARD)
        codes = torch.full((1, n, cfg.code_row_bytes), 0xEE, dtype=torch.uint8, device="cuda")
        A.adamas_encode_keys(cfg, torch.from_numpy(bits_of(x).view(np.int16)).view(torch.bfloat16).cuda()[None], codes, 0, n)
        with oracle.head_dim(d):
            ref = oracle.encode_bits(bits_of(x), thr, bits, hadamard=hadamard)[1]
        assert np.array_equal(codes.cpu().numpy()[0], ref)
