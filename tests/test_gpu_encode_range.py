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


@pytest.mark.parametrize("bits,d", [(4, 96), (4, 128), (4, 256), (4, 512), (4, 1024), (2, 256), (2, 4096)])
def test_dimensions_that_fill_the_sorted_table(bits, d):
    """As many positive magnitudes as the table holds, equal ones among them, zeros, and few dimensions (runs too short to
    end early): the oracle's codes."""
    from paper_2601_07048_amd import jx

    rng = np.random.default_rng(d + bits)
    n = 40
    r = rng.standard_normal((n, d)).astype(np.float32)
    r[1] = 1.0
    r[2] = np.sign(r[2]) * rng.integers(1, 4, d)
    r[3, : d // 2] = 0.0
    r[4] = 0.0
    r[5] = np.float32(2.0) ** rng.integers(-20, 20, d)
    g = jx.Index(d, jx.U8, 8, 8, 1.2, capacity=n, quant_bits=bits)
    g.import_graph(dev(np.zeros((n, d), np.uint8)), dev(np.full((n, 8), jx.NONE, np.uint32)), 0)
    g.quantize(bits, dev(np.eye(d, dtype=np.float32)), dev(np.zeros(d, np.float32)), rule=jx.RULE_MAXCOS)
    codes, _ = g.encode_rotated(dev(r))
    assert np.array_equal(codes.cpu().numpy(), oracle.rabitq_encode(r, bits, oracle.RULE_MAXCOS)[0])
