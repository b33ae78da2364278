"""The decomposition's kernels at the edges of their tiles: one row tile, rows that end inside a tile of 64 and of 128, and more
rows than 64 parts of the Gram matrix hold in one stage each."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn", [(32, 256), (160, 512), (352, 1280), (8224, 256), (256, 8448)])
def test_factors_and_signs_at_tile_edges(out, inn):
    import torch
    import paper_2410_23918_amd as B
    rng = np.random.default_rng(out + inn)
    w = (0.02 * rng.standard_normal((out, inn))).astype(np.float32)
    s = np.exp(0.5 * rng.standard_normal(inn)).astype(np.float32)
    sw, U, V = B.decompose(torch.from_numpy(w).to("cuda:0"), s, 2)
    torch.cuda.synchronize()
    bits = np.unpackbits(sw.cpu().numpy().view(np.uint8).reshape(2, out, inn // 8), axis=2, bitorder="little").astype(bool)
    U, V = U.cpu().numpy().astype(np.float64), V.cpu().numpy().astype(np.float64)
    R = (w * s[None, :]).astype(np.float64)   # the product rounded to fp32, as on the device
    for i in range(2):
        # the device's later residuals carry one fp32 rounding per element: signs may differ within that of zero
        differ = bits[i] != ~(R < 0.0)
        assert not differ.any() if i == 0 else np.abs(R[differ]).max(initial=0.0) <= 1e-6 * np.abs(w * s).max()
        sv = np.linalg.svd(np.abs(R), compute_uv=False)
        best = np.sqrt(np.sum(np.square(sv[16:])))
        m = U[i] @ V[i].T
        err = np.linalg.norm(np.abs(R) - m)
        # no rank-16 matrix is closer than `best`; fp16 factors add 2^-11 of the leading part at most, and 16 rounds with 16 spare
        # columns leave 1e-3 of the truncation error
        assert best * (1 - 1e-9) <= err <= np.hypot(best * (1 + 1e-3), 2.0 ** -11 * np.linalg.norm(m)) + 1e-12
        R = R - np.where(bits[i], m, -m)
