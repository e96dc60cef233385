"""The resident-factor decode and residual passes (bf16 caches, d >= 64) at the edges of their
tiles: lengths around 32-token tiles and 256-token rounds, every code width and the group sizes
one row's scales allow, ranks off the multiples of 8, and a group size that takes the staged kernel.

Codes are compared stage-wise (the oracle's quantiser on the GPU's own X~, one level on at most
1e-4 of the entries plus one entry); decoded rows with the oracle's decode of the same blob within
one bf16 rounding (2^-8 of the entry) plus fp32 sums (1e-5 of the cell's rms).
"""
import numpy as np
import pytest
import torch

import paper_2607_12550_amd as J
from gpu_util import blob_bytes, compress, ctx, decompress, device_cells, note, workspace
from oracle import pipeline as opl
from oracle.philox import rotation_signs
from oracle.residual import quantize, rotate
from oracle.rope import rope

pytestmark = pytest.mark.gpu

#     d   m  T    r_T  r_d bits group
CASES = [(128, 2, 33, 8, 8, 8, 64), (128, 3, 257, 40, 40, 4, 128), (128, 2, 300, 136, 72, 2, 32),
         (64, 3, 31, 16, 16, 2, 64), (64, 2, 289, 24, 8, 8, 16), (64, 4, 70, 20, 12, 4, 32),
         (128, 1, 1, 1, 8, 4, 64), (128, 2, 100, 24, 16, 4, 16), (128, 2, 64, 0, 0, 8, 64)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "d%d_m%d_T%d_r%d_%d_b%d_g%d" % c)
def test_codes_and_decoded_rows(case):
    d, m, T, rT, rd, bits, group = case
    rng = np.random.default_rng(T)
    X = rng.standard_normal((m, T, 8)) @ rng.standard_normal((8, d)) + 0.3 * rng.standard_normal((m, T, d))
    xs, ex, desc = device_cells([X], "bf16")
    blobs, _ = compress(xs, desc, [J.Params(rT, rd, bits, group, J.JOLT_FACTOR_F16, 0, 9)])
    Xt = torch.empty((m, T, d), device="cuda")
    J.jolt_debug_export(ctx(), 2, 0, Xt)
    Xt = Xt.cpu().numpy().astype(np.float64)
    b = blob_bytes(blobs[0])
    got = opl.read_blob(b)
    codes, scales = quantize(rotate(ex[0] - Xt, rotation_signs(9, d)), bits, group)
    diff = np.abs(np.asarray(got["codes"], dtype=np.int64).reshape(-1) - np.asarray(codes, dtype=np.int64).reshape(-1))
    assert diff.max() <= 1 and (diff > 0).sum() <= 1 + 1e-4 * diff.size
    np.testing.assert_allclose(np.asarray(got["scales"], dtype=np.float64).reshape(-1), np.asarray(scales, dtype=np.float64).reshape(-1), rtol=2e-3)
    want = opl.decode_blob(b)
    out = decompress(blobs, desc, "bf16")[0]
    rms = np.sqrt((want ** 2).mean())
    assert (np.abs(out - want) <= 2.0 ** -8 * np.abs(want) + 1e-5 * rms).all()


@pytest.mark.parametrize("d, T, bits", [(64, 65, 8), (128, 128, 4)])
def test_short_slices_in_one_call_or_alone(d, T, bits):
    """512 slices of at most 128 tokens are decoded by the staged kernel, those of one cell alone by
    the resident one: the same bits."""
    n, m = 8, 64
    rng = np.random.default_rng(d)
    cells = [rng.standard_normal((m, T, 8)) @ rng.standard_normal((8, d)) + 0.3 * rng.standard_normal((m, T, d)) for _ in range(n)]
    xs, ex, desc = device_cells(cells, "bf16")
    blobs, _ = compress(xs, desc, [J.Params(24, 16, bits, 32, J.JOLT_FACTOR_F16, 0, i) for i in range(n)])
    both = decompress(blobs, desc, "bf16")
    for i in (0, n - 1):
        assert np.array_equal(both[i], decompress(blobs[i:i + 1], desc, "bf16")[0])


@pytest.mark.parametrize("d, T, offset", [(64, 33, 0), (64, 289, 100000), (128, 33, 1000000), (128, 289, 123457)])
def test_rope_at_large_positions(d, T, offset):
    """Rows decoded with RoPE against the oracle's rotation of its decode, ragged lengths and large
    positions (the angle is reduced in fp64: its error stays below 1e-9 at 1e6)."""
    rng = np.random.default_rng(T + d)
    X = rng.standard_normal((4, T, 8)) @ rng.standard_normal((8, d)) + 0.3 * rng.standard_normal((4, T, d))
    xs, ex, desc = device_cells([X], "bf16")
    blobs, _ = compress(xs, desc, [J.Params(16, 16, 4, 32, J.JOLT_FACTOR_F16, 0, 5)])
    want = rope(opl.decode_blob(blob_bytes(blobs[0])), 1e6, np.arange(T) + float(offset))
    out = torch.empty((4, T, d), dtype=torch.bfloat16, device="cuda")
    note("jolt_decompress_rope d", d, "T", T, "offset", offset)
    J.jolt_decompress(ctx(), blobs, desc, [out], workspace(desc, 1), rope=(1e6, offset))
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    rms = np.sqrt((want ** 2).mean())
    assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 1e-5 * rms).all()
