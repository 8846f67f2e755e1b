"""Mask compaction at the sizes where its kernels change form (one workgroup a head, 1 to 5 steps of 1,024 columns a row,
every alignment of a row), against the mask itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from tests.gpu_util import csr_matches_mask   # noqa: E402


@pytest.mark.parametrize("mb", [1, 15, 16, 17, 127, 128, 129, 1009, 1010, 2033, 2034, 3057, 3058, 4081, 4082])
def test_compact_edges(mb):
    import paper_2609_34814_amd as W
    heads = 3 if mb < 2000 else 1
    rng = np.random.default_rng(mb)
    mask = (rng.random((1, heads, mb, mb)) < 0.1).astype(np.uint8) * rng.integers(1, 256, (1, heads, mb, mb), dtype=np.uint8)
    mask[0, 0, 0] = 255                 # a full row, an empty one and the row's two ends
    if mb > 2:
        mask[0, 0, 1] = 0
        mask[0, 0, 2] = 0
        mask[0, 0, 2, [0, mb - 1]] = 128
    # an odd start address: rows begin at every byte of a 16-byte chunk
    buf = torch.zeros(mask.size + 16, dtype=torch.uint8, device="cuda")
    for off in (0, 5):
        md = buf[off:off + mask.size].view(mask.shape)
        md.copy_(torch.from_numpy(mask))
        rp, ci = W.compact_mask(md, seq_len=64 * mb, block=64)
        rp, ci = rp.cpu().numpy(), ci.cpu().numpy()
        for h in range(heads):
            assert csr_matches_mask(mask[0, h], rp[0, h], ci[h * mb * mb:(h + 1) * mb * mb]), (mb, h, off)
