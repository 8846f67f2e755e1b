"""The permutation at the sizes where its kernels change form, bit for bit against the oracle: workgroups of 256, 512
and 1,024 threads, rank and bitonic sorts, two and four keys a thread, word groups, slices of a head."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import skip as S   # noqa: E402
from tests.test_gpu_parity import _perm_case   # noqa: E402
from workloads import make_mask   # noqa: E402
from workloads.gen import custom   # noqa: E402


def _wl(blocks, heads=1, seed=31):
    # 16 tokens a row of blocks' worth of grid: one frame per four blocks, the last block ragged
    return custom(f"forms{blocks}", heads=heads, head_dim=64, block=64, grid=(max(1, -(-blocks // 4)), 16, 16),
                  seq_len=64 * blocks - 3, seed=seed, rule=dict(kind="radius", rt=2, rs=1, g=3))


@pytest.mark.parametrize("blocks", [128, 129, 256, 257, 512, 513])
@pytest.mark.parametrize("mode", [S.SKIP_NEVER, S.SKIP_AUTO])
def test_one_workgroup_forms(blocks, mode):
    wl = _wl(blocks, heads=2)
    _perm_case(wl, make_mask(wl), wave=7, n_xcd=8, mode=mode, iters=3)


@pytest.mark.parametrize("blocks", [2048, 2049])
def test_sliced_form(blocks):
    wl = _wl(blocks)
    _perm_case(wl, make_mask(wl), wave=64, n_xcd=8, mode=S.SKIP_NEVER, iters=2)


@pytest.mark.parametrize("blocks", [100, 300, 1100])
def test_rows_of_one_angle_and_many_heads(blocks):
    """Rows of five kinds only (equal rows have equal angles and keep their order), over so many heads that a head has
    one slice; one head has equal rows throughout (degenerate), one is empty."""
    heads = 300 if blocks > 1024 else 3
    wl = _wl(blocks, heads=3)
    rng = np.random.default_rng(blocks)
    kinds = rng.random((5, blocks)) < 0.3
    kinds[:, 0] = True
    mask = np.stack([kinds[rng.integers(0, 5, blocks)], np.tile(kinds[0], (blocks, 1)),
                     np.zeros((blocks, blocks), dtype=bool)]).astype(np.uint8)[None]
    perm, _ = _perm_case(wl, mask, wave=64, n_xcd=4, mode=S.SKIP_NEVER, iters=2)
    if heads > 3:  # the same three heads, a hundred times over (the seed of a head's start block is its index)
        import paper_2609_34814_amd as W
        big = torch.from_numpy(np.tile(mask, (1, heads // 3, 1, 1))).cuda()
        got, seg, _ = W.build_permutation(big, seq_len=wl.seq_len, block=64, head_dim=64, wave=64, n_xcd=4, skip="never",
                                          iters=2)
        assert np.array_equal(got[:, :3].cpu().numpy(), perm)
        srt = got.sort(dim=-1).values
        assert bool((srt == torch.arange(wl.mb, device="cuda", dtype=torch.int32)).all())


def test_wave_sizes_do_not_follow_the_kernel():
    """The default wave is part of what a default permutation is: fixed per shape (32 compute units per XCD)."""
    import paper_2609_34814_amd as W
    cus = torch.cuda.get_device_properties(0).multi_processor_count // 8
    want = {(64, 64): 6, (64, 128): 2, (128, 64): 4, (128, 128): 2}
    assert {k: W.wave_size(*k) for k in want} == {k: cus * v for k, v in want.items()}
