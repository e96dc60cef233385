"""The chunk pass of decode attention at the edges of its dispatch and of its tiles.

The matrix-core pass takes fp16 factors with ranks in multiples of 8 and quantiser groups of at
least 32 features, everything else the vector pass; both are compared with the oracle's softmax
attention over the oracle's decode.  The operands that are split carry at least 24 bits and all
sums are fp32 over at most a few thousand terms, so every output entry is within
sqrt(2000) * 2^-22 ~ 1e-5 of the norm of its head's output.
"""
import numpy as np
import pytest

import paper_2607_12550_amd as J  # noqa: F401  (loads the library)
from oracle import attention as oat, pipeline as opl
from test_gpu_attend import _cell, _oracle_blob, _run

pytestmark = pytest.mark.gpu
TOL = 1e-5

#     d    H  rep  T    group  keys (r_T, r_d, bits)  values (r_T, r_d, bits)
CASES = [
    (128, 2, 4, 129, 64, (24, 16, 8), (40, 24, 4)),      # ragged last tile, rank steps not full
    (128, 2, 8, 65, 32, (32, 8, 4), (16, 8, 2)),         # two query tiles, four groups a row
    (128, 1, 5, 63, 128, (8, 8, 2), (8, 8, 8)),          # five heads, one group a row
    (64, 3, 3, 200, 64, (64, 16, 8), (72, 16, 8)),       # d = 64
    (64, 2, 1, 64, 32, (0, 0, 4), (16, 16, 0)),          # no key backbone, no value residual
    (32, 2, 2, 100, 32, (40, 8, 2), (24, 16, 4)),        # d = 32: one step a row
    (128, 2, 2, 700, 64, (296, 16, 4), (264, 24, 4)),    # ranks past the registers and tiles of small ones
    (128, 2, 8, 600, 64, (16, 8, 4), (512, 16, 2)),      # largest value rank
    (128, 2, 2, 100, 16, (24, 16, 4), (16, 16, 4)),      # groups of 16: vector pass
    (128, 2, 2, 100, 64, (20, 16, 4), (13, 10, 4)),      # ranks off the multiples of 8: vector pass
    (64, 2, 4, 1, 64, (0, 0, 8), (1, 8, 2)),             # one token
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "d%d_H%d_rep%d_T%d_g%d_k%d_v%d" % (*c[:5], c[5][0], c[6][0]))
def test_chunk_pass_edges(case):
    d, H, rep, T, group, kp, vp = case
    rng = np.random.default_rng(11)
    K, V = _cell(rng, 2 * H, T, d, 1.5), _cell(rng, 2 * H, T, d, 0.7)
    if max(kp[0], vp[0]) > 64:      # enough energy past the 16 shared directions for the ranks asked
        K, V = K + 0.2 * rng.standard_normal(K.shape), V + 0.2 * rng.standard_normal(V.shape)
    blobs = [_oracle_blob(X, H, *p, group, 5 + i) for i, (X, p) in enumerate(((K, kp), (V, vp)))]
    Q = rng.standard_normal((2, rep * H, d))
    got = _run([blobs[0]] * 2, [blobs[1]] * 2, [1, 0], Q, d)
    K, V = opl.decode_blob(blobs[0]), opl.decode_blob(blobs[1])
    Q = Q.astype(np.float32).astype(np.float64)
    for i, layer in enumerate((1, 0)):
        want = oat.attend(K, V, layer, H, Q[i], 1.0 / np.sqrt(d))
        for j in range(rep * H):
            assert np.abs(got[i, j] - want[j]).max() <= TOL * np.linalg.norm(want[j]), (i, j)


# calls of enough workgroups that a key-value head's query heads share a combine workgroup (four, five
# of eight, eight of them), the last with value ranks past 256 on the matrix cores
@pytest.mark.parametrize("d, rep, T, v_rT", [(128, 4, 70, 16), (64, 5, 70, 24), (64, 8, 1024, 264)])
def test_many_items(d, rep, T, v_rT):
    H, n = 8, 32
    rng = np.random.default_rng(12)
    K, V = _cell(rng, H, T, d, 1.5), _cell(rng, H, T, d, 0.7) + 0.2 * rng.standard_normal((H, T, d))
    kb, vb = _oracle_blob(K, H, 24, 16, 4, 32, 5), _oracle_blob(V, H, v_rT, 24, 4, 32, 6)
    Q = rng.standard_normal((n, rep * H, d))
    got = _run([kb] * n, [vb] * n, [0] * n, Q, d)
    K, V = opl.decode_blob(kb), opl.decode_blob(vb)
    Q = Q.astype(np.float32).astype(np.float64)
    for i in range(0, n, 5):
        want = oat.attend(K, V, 0, H, Q[i], 1.0 / np.sqrt(d))
        for j in range(rep * H):
            assert np.abs(got[i, j] - want[j]).max() <= TOL * np.linalg.norm(want[j]), (i, j)
