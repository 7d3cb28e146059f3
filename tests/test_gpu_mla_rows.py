"""The latent-KV kernel for few query rows (up to 32 per sequence) against the oracle."""
import numpy as np
import pytest

import oracle
from workloads import bf16_to_f32
from test_gpu_mla import DV, SCALE, _case, _default_partition, gpu_mla      # noqa: F401  (the fixture resets the knobs)

pytestmark = pytest.mark.gpu


# rows 1, 15, 16 (one tile), 17, 32 (two), 33 (the kernel for more rows); lengths around the 32-key block, unsplit
# sequences and sequences of many segments; one bf16 per weight where the caller asks for it
@pytest.mark.parametrize("T,H", [(1, 1), (3, 5), (2, 8), (1, 17), (16, 2), (3, 11)])
@pytest.mark.parametrize("pieces,pv_mode,scale_up", [(0, 0, 1.0), (8, 0, 16.0), (37, 2, 1.0), (2048, 1, 4.0)])
def test_few_rows(T, H, pieces, pv_mode, scale_up):
    import paper_2510_14686_amd as xa
    from gpu_util import TOL_LSE, TOL_REL_L2, assert_parity, errors
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
    lens = [max(T, n) for n in (1, 31, 32, 33, 63, 65, 97, 700, 2049)]
    q, cs = _case(300 + T, lens, T, H)
    scale = float(np.float32(SCALE * scale_up))
    out_bits, lse = gpu_mla(q, cs, lens, scale)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, scale)
    what = "T=%d H=%d pieces=%d" % (T, H, pieces)
    if scale_up == 1.0:
        assert_parity(out_bits, lse, ref_out, ref_lse, what)
        return
    # One key can carry a row here, so single outputs reach the largest of the values (|v| up to 5): the
    # absolute bar presumes |out| < 4.  Element by element instead: rounding to bf16 (half an ulp is at most
    # 2^-8 of the value) and the fp16 partial rows (2^-11 of values up to 5, weights summing to 1).
    max_abs, rel_rows, _, lse_err = errors(out_bits, lse, ref_out, ref_lse)
    diff = np.abs(bf16_to_f32(out_bits).astype(np.float64).reshape(ref_out.shape) - ref_out)
    assert np.all(diff <= 2.0 ** -8 * np.abs(ref_out) + 5 * 2.0 ** -11), what
    assert rel_rows <= TOL_REL_L2 and lse_err <= TOL_LSE, what
