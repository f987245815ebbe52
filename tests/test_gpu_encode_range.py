"""The max-cosine encoder rules breakpoints out with float32 estimates: vectors at both ends of the float32 range, and one
coordinate far above the others, give the oracle's codes."""
import numpy as np
import pytest

import oracle
from gpu_common import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("scale", [1e-37, 1e-20, 1.0, 1e20, 1e35])
def test_scales(bits, scale):
    from paper_2601_07048_amd import jx

    n, d = 60, 96
    x = np.random.default_rng(bits).standard_normal((n, d))
    x[1, 0] = 900.0
    x[2] = np.exp2(np.arange(d) / 8.0 - 6.0)
    x[3, :90] = 1e-3
    r = (x * scale).astype(np.float32)
    g = jx.Index(d, jx.F32, 8, 8, 1.2, capacity=n, quant_bits=bits)
    g.import_graph(dev(x.astype(np.float32)), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(bits, dev(np.eye(d, dtype=np.float32)), dev(np.zeros(d, np.float32)), rule=jx.RULE_MAXCOS)
    codes, _ = g.encode_rotated(dev(r))
    assert np.array_equal(codes.cpu().numpy(), oracle.rabitq_encode(r, bits, oracle.RULE_MAXCOS)[0])
