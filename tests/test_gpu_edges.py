"""Kernels at the sizes where their work split can go wrong: edges of
vectors, tiles and groups, remainders, views that start off a vector
boundary.  Same oracle and bounds as the kernel parity tests."""
import numpy as np
import pytest

from oracle import quant

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
DEV = "cuda"


def _srp():
    import paper_2106_12060_amd as srp
    return srp


def off_boundary(X, elements):
    """Contiguous device copy of X that starts `elements` past an allocation."""
    t = torch.from_numpy(np.ascontiguousarray(X))
    buf = torch.zeros(t.numel() + elements, dtype=t.dtype, device=DEV)
    buf[elements:] = t.reshape(-1).to(DEV)
    return buf[elements:].view(t.shape)


# groups of M = 4 ceil(256 / d) rows: fewer rows than a group, a remainder of
# rows, one column, widths around the 256-thread workgroup
@pytest.mark.parametrize("n,d,off", [(3, 60, 0), (1, 1, 1), (2049, 1, 0), (517, 3, 1), (1031, 255, 2),
                                     (64, 256, 0), (403, 257, 3), (4099, 131, 1)])
def test_staging_group_edges(n, d, off):
    srp = _srp()
    rng = np.random.default_rng(100 * n + d)
    grid = np.concatenate([quant._FP8_VALS, (quant._FP8_VALS[1:] + quant._FP8_VALS[:-1]) / 2])   # values and ties
    X = (rng.choice(grid, size=(n, d)) * rng.choice([-1.0, 1.0], size=(n, d)) *
         2.0 ** rng.integers(-3, 4, size=d)[None, :]).astype(np.float32)
    X[rng.random((n, d)) < 0.3] *= np.float32(1 + 2.0 ** -20)
    Xd = off_boundary(X, off)
    codes, scales = srp.srp_stage_fp8(Xd)
    ref, sc = quant.fp8_stage(X)
    np.testing.assert_array_equal(scales.cpu().numpy(), sc)
    np.testing.assert_array_equal(codes.cpu().numpy(), ref)
    np.testing.assert_array_equal(srp.srp_stage_bf16(Xd).float().cpu().numpy(), quant.bf16_round(X))
    Xb = off_boundary(quant.bf16_round(X).astype(np.float32), 0).to(torch.bfloat16)
    codes, scales = srp.srp_stage_fp8(Xb)
    ref, sc = quant.fp8_stage(Xb.double().cpu().numpy())
    np.testing.assert_array_equal(scales.cpu().numpy(), sc)
    np.testing.assert_array_equal(codes.cpu().numpy(), ref)
