"""Rows computed in chunks by several workgroups (launches whose longest row would outlast the rest): the
edges of the split rule against the oracle, for every head_dim and block."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import attention as A   # noqa: E402
from tests.gpu_util import bf16_dev, compare_blocks, dev_f64, u8_dev   # noqa: E402
from workloads.gen import custom, make_qkv   # noqa: E402

MIN_L = 12   # the shortest L: on launches this small, rows of more kept blocks are split
WGS = {(64, 64): 6, (64, 128): 2, (128, 64): 4, (128, 128): 2}   # workgroups on a compute unit


def _plan(counts, d, block):
    """(chunks, L, first L) of the split rule for the rows' kept blocks [heads][mb]."""
    n, mb = np.asarray(counts).ravel().astype(np.int64), np.asarray(counts).shape[-1]
    slots = torch.cuda.get_device_properties(0).multi_processor_count * WGS[d, block]
    cap = min((32 << 20) // (4 * block * (d + 2)), n.size * -(-mb // MIN_L))
    kept = int(n.sum())
    L = first = max(MIN_L, -(-(kept * 5 // 4) // slots))
    while L < mb:
        chunks = int((-(-n[n > L] // L)).sum())
        use = chunks if chunks <= cap else 0
        merge, fixed = (24 if d == 64 else 16, 4) if block == 64 else (16, 0)
        if slots * (9 * int(n.max()) - 5 * L - 10 * fixed) <= 10 * (kept + merge * use):
            break
        if chunks <= cap:
            return chunks, L, first
        L += (L + 1) // 2
    return 0, L, first


def _planned(q, k, v, mask, block):
    """(O, LSE, chunks, L): a call in a workspace of its own, from which the plan is read back."""
    import ctypes
    import paper_2609_34814_amd as W
    from paper_2609_34814_amd import _lib as L
    b, h, n, d = q.shape
    shape, size = W.shape_of(b, h, n, d, block), ctypes.c_size_t(0)
    assert L.load().wa_attn_workspace_size(ctypes.byref(shape), ctypes.byref(size)) == 0
    ws = torch.zeros(W.attn_workspace_size(shape), dtype=torch.uint8, device="cuda")
    o, lse = W.sparse_attn(q, k, v, mask, block=block, return_lse=True, workspace=ws)
    chunks, longest = ws[size.value:size.value + 8].view(torch.int32).tolist()
    return o, lse, chunks, longest


def _mask(heads, mb, rng):
    """Row lengths around multiples of L, a full row (it holds the ragged last block), an empty row, the
    last block alone, and the diagonal elsewhere."""
    m = np.zeros((1, heads, mb, mb), dtype=np.uint8)
    for h in range(heads):
        m[0, h] = np.eye(mb, dtype=np.uint8)
        for row, n in ((1, MIN_L - 1), (2, MIN_L), (3, MIN_L + 1), (4, 2 * MIN_L), (5, 2 * MIN_L + 1), (6, mb)):
            m[0, h, row] = 0
            m[0, h, row, np.sort(rng.permutation(mb)[:n])] = 1
        m[0, h, 7] = 0
        m[0, h, 8] = 0
        m[0, h, 8, mb - 1] = 1
    return m


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("scale_k", [1, 32])
def test_split_rows_vs_oracle(d, block, scale_k):
    """scale_k = 32: K of the upper blocks scaled, so that chunks recompute against their exact maximum and
    chunks of one row have maxima far apart."""
    import paper_2609_34814_amd as W
    mb, heads = 41, 2
    wl = custom("split", heads=heads, head_dim=d, block=block, grid=(1, 1, mb * block), seq_len=mb * block - 7, seed=21)
    rng = np.random.default_rng(d + block)
    mask = _mask(heads, mb, rng)
    q, k, v = make_qkv(wl)
    kd = bf16_dev(k).float()
    kd[:, :, mb // 2 * block:] *= scale_k      # exact: a power of two
    kd = kd.to(torch.bfloat16)
    k_bits = kd.view(torch.int16).cpu().numpy().view(np.uint16)
    qd, vd, md = bf16_dev(q), bf16_dev(v), u8_dev(mask)
    o, lse, chunks, longest = _planned(qd, kd, vd, md, block)
    assert (chunks, longest) == _plan(mask[0].sum(-1), d, block)[:2] == (heads * 11, MIN_L)   # 2 + 2 + 3 + 4 a head
    ref_o, ref_lse = A.block_sparse_attention(q, k_bits, v, mask, block)
    ref = {}
    for h in range(heads):
        for i in range(mb):
            lo, hi = A.block_token_range(i, block, wl.seq_len)
            ref[(0, h, i)] = (ref_o[0, h, lo:hi], ref_lse[0, h, lo:hi])
    st = compare_blocks(dev_f64(o), ref, block, wl.seq_len, lse.cpu().numpy().astype(np.float64))
    print("split", d, block, scale_k, st)
    # bf16 probabilities and output: 2 * 2^-9 relative each; one key dominates short rows, so the
    # absolute bar scales with max|V|
    assert st["max_abs"] <= 4 * 2.0 ** -9 * float(np.abs(A.bf16_to_f64(v)).max()), st
    assert st["rel_rms"] <= 1e-2 and st["lse"] <= 1e-3, st

    # the split follows from the lists alone: any order, queue count and entry point gives the same bytes
    rp, ci = W.compact_mask(md, seq_len=wl.seq_len, block=block, head_dim=d)
    vt = W.transpose_v(vd, block=block)
    perm = torch.from_numpy(np.stack([rng.permutation(mb) for _ in range(heads)])[None].astype(np.int32)).cuda()
    for p, nx, order in ((perm, 8, "in-order"), (perm, 1, "interleaved"), (None, 64, "in-order")):
        o2, l2 = W.sparse_attn_vt(qd, kd, vt, rp, ci, p, block=block, n_xcd=nx, head_order=order, return_lse=True)
        assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, l2)
        out, l3 = torch.full_like(o, float("nan")), torch.full_like(lse, float("nan"))
        W.sparse_attn_vt_noalloc(qd, kd, vt, rp, ci, p, block=block, n_xcd=nx, head_order=order, out=out, lse=l3)
        assert torch.equal(o.view(torch.int16), out.view(torch.int16)) and torch.equal(lse, l3)

    # a split row that no slot names keeps its old contents, and an invalid index in a chunk is reported
    bad = torch.arange(mb, dtype=torch.int32, device="cuda").repeat(1, heads, 1).contiguous()
    bad[0, 0, 6] = mb
    ci2 = ci.clone()
    ci2[mb * mb + int(rp[0, 1, 7].item()) - 1] = -3
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    out = torch.full_like(o, float("nan"))
    W.sparse_attn_vt(qd, kd, vt, rp, ci2, bad, block=block, out=out, status=status)
    lo, hi = A.block_token_range(6, block, wl.seq_len)
    assert int(status.item()) == 3
    assert bool(torch.isnan(out[0, 0, lo:hi].float()).all())
    out[0, 0, lo:hi] = o[0, 0, lo:hi]
    out[0, 1, lo:hi] = o[0, 1, lo:hi]
    assert torch.equal(o.view(torch.int16), out.view(torch.int16))


def _rows_of(counts, rng):
    """Mask with the given numbers of kept blocks [heads][mb], at random."""
    heads, mb = counts.shape
    m = np.zeros((1, heads, mb, mb), dtype=np.uint8)
    for h in range(heads):
        for i in range(mb):
            m[0, h, i, rng.permutation(mb)[:counts[h, i]]] = 1
    return m


def _against_oracle(wl, mask, picks, block, plan):
    """A call whose chunks and L are those of `plan`, compared on the picked rows."""
    q, k, v = make_qkv(wl)
    o, lse, chunks, longest = _planned(bf16_dev(q), bf16_dev(k), bf16_dev(v), u8_dev(mask), block)
    assert (chunks, longest) == plan
    assert bool(torch.isfinite(o.float()).all()) and bool(torch.isfinite(lse).all())
    ref = A.block_sparse_attention_rows(q, k, v, mask, block, picks)
    st = compare_blocks(dev_f64(o), ref, block, wl.seq_len, lse.cpu().numpy().astype(np.float64))
    assert st["max_abs"] <= 4 * 2.0 ** -9 * float(np.abs(A.bf16_to_f64(v)).max()), st
    assert st["rel_rms"] <= 1e-2 and st["lse"] <= 1e-3, st


def test_split_rows_up_to_the_tile_limit():
    """More chunks than tiles (d 128, block 128: 504): L grows until they fit, with 186 rows in two chunks."""
    mb, heads, d, block = 128, 2, 128, 128
    wl = custom("split-limit", heads=heads, head_dim=d, block=block, grid=(1, 1, mb * block), seed=22)
    rng = np.random.default_rng(22)
    counts = np.ones(heads * mb, dtype=np.int64)
    rows = rng.permutation(heads * mb)[:186]
    counts[rows[:180]], counts[rows[180:]] = 100, mb
    counts = counts.reshape(heads, mb)
    chunks, longest, first = _plan(counts, d, block)
    limit = (32 << 20) // (4 * block * (d + 2))
    assert int((-(-counts[counts > first] // first)).sum()) > limit >= chunks > 0 and longest > first
    picks = [(0, int(r) // mb, int(r) % mb) for r in rows[[0, 1, 90, 179, 180, 185]]]
    _against_oracle(wl, _rows_of(counts, rng), picks, block, (chunks, longest))


@pytest.mark.parametrize("d,block,heads", [(64, 64, 8), (64, 128, 3)])
def test_more_chunks_than_workgroups(d, block, heads):
    """Rows of 30 blocks in two chunks each, a few full rows and one row of one block a head: more chunks than the device
    holds workgroups (the shapes whose tile limit allows it), so the chunks past the first of each workgroup come
    from the shards' counters."""
    mb = 100
    wl = custom("split-many", heads=heads, head_dim=d, block=block, grid=(1, 1, mb * block), seed=23)
    rng = np.random.default_rng(d + block)
    counts = np.full((heads, mb), 30)
    counts[:, 0], counts[:, mb - 1], counts[0, 7], counts[1, 9] = 1, mb, mb, mb
    chunks, longest, _ = _plan(counts, d, block)
    assert chunks > torch.cuda.get_device_properties(0).multi_processor_count * WGS[d, block] and longest < 30
    picks = [(0, h, i) for h in range(heads) for i in (0, 1, h + 5, mb - 1)] + [(0, 0, 7), (0, 1, 9)]
    _against_oracle(wl, _rows_of(counts, rng), picks, block, (chunks, longest))


@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_split_rows_with_scores_of_minus_infinity(d, block):
    """Chunks whose scores are all -inf (keys of the lower blocks hold -inf against positive queries) add nothing to
    a row that has finite ones; a row of -inf alone has no value (NaN, lse -inf), split or not; NaN scores stay NaN."""
    import paper_2609_34814_amd as W
    mb = 3 * MIN_L + 5
    n, low = mb * block - 7, 2 * MIN_L * block
    g = torch.Generator().manual_seed(d + block)
    q, k, v = (torch.randn(1, 1, n, d, generator=g).to(torch.bfloat16) for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 0.5
    k[:, :, :low, 0] = -float("inf")
    k[:, :, low + block, 1] = float("nan")
    mask = torch.zeros(1, 1, mb, mb, dtype=torch.uint8)
    mask[0, 0, :, :] = torch.eye(mb, dtype=torch.uint8)
    mask[0, 0, 1, :] = 1
    mask[0, 0, 1, low // block + 1] = 0        # split, -inf in its first chunks, finite in its last
    mask[0, 0, 2, : low // block] = 1          # split, -inf alone
    mask[0, 0, 3, :] = 1                       # split, with the NaN key
    mask[0, 0, 4, [4, mb - 1]] = 1             # not split, -inf then finite
    o, lse = W.sparse_attn(q.cuda(), k.cuda(), v.cuda(), mask.cuda(), block=block, return_lse=True)
    o, lse = o.double().cpu()[0, 0], lse.double().cpu()[0, 0]
    keep = mask[0, 0].bool().repeat_interleave(block, 0).repeat_interleave(block, 1)[:n, :n]
    for row in (1, 4):
        t = slice(row * block, (row + 1) * block)
        keys = keep[row * block]
        s = q[0, 0, t].double() @ k[0, 0, keys].double().T / d ** 0.5
        want = torch.softmax(s, -1) @ v[0, 0, keys].double()
        # bf16 probabilities and output: 2 * 2^-9 relative each, of values up to max|V|
        assert float((o[t] - want).abs().max()) <= 4 * 2.0 ** -9 * float(v.double().abs().max()), row
        assert float((lse[t] - torch.logsumexp(s, -1)).abs().max()) <= 1e-3, row
    for row in (2, 3):
        assert bool(torch.isnan(o[row * block:(row + 1) * block]).all()), row
    assert bool(torch.isneginf(lse[2 * block:3 * block]).all())


@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_split_rows_take_the_reference_of_the_unsplit_row(d, block):
    """A head alone (its rows split) and the same head among 63 full ones (L above M_B: no row split). Both take their
    probabilities against the row's first block, so they differ by the order of float32 sums: a few 1e-6 of
    a value, which moves one bf16 rounding in some thousand (2^-9 apart) by one step. Keys of a chunk whose scores lie far
    below the first block's have probability 0 in both, also with values near the largest float."""
    import paper_2609_34814_amd as W
    mb, n = 41, 41 * block - 7
    g = torch.Generator(device="cuda").manual_seed(d + block)
    q, k, v = (torch.randn(1, 64, n, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    far = slice((mb - 8) * block, (mb - 4) * block)
    q[0, 0, 6 * block:7 * block, 0] = 8.0
    k[0, 0, far, 0] = -1024.0
    v[0, 0, far] = 3e38
    mask = torch.ones(1, 64, mb, mb, dtype=torch.uint8, device="cuda")
    mask[0, 0] = u8_dev(_mask(1, mb, np.random.default_rng(d + block))[0, 0])
    mask[0, 0, :, mb - 8:mb - 4] = 0
    mask[0, 0, 6] = 1
    whole, lse = W.sparse_attn(q, k, v, mask, block=block, return_lse=True)
    split, lse_s = W.sparse_attn(*(x[:, :1].contiguous() for x in (q, k, v)), mask[:, :1].contiguous(), block=block,
                                 return_lse=True)
    a, b = whole[0, 0].float(), split[0, 0].float()
    assert bool(torch.isfinite(a).all()) and bool(torch.isfinite(b).all())
    rows = torch.zeros(n, dtype=torch.bool, device="cuda")
    for r in (3, 4, 5, 6):     # more than MIN_L blocks
        rows[r * block:(r + 1) * block] = True
    assert torch.equal(a[~rows], b[~rows])
    share = float((a[rows] != b[rows]).float().mean())
    rel = float((a[rows] - b[rows]).norm() / a[rows].norm())
    print("split against whole", d, block, share, rel)
    assert share <= 1e-2 and rel <= 2e-4, (share, rel)
    fin = torch.isfinite(lse[0, 0])
    assert torch.equal(fin, torch.isfinite(lse_s[0, 0]))
    assert float((lse[0, 0][fin] - lse_s[0, 0][fin]).abs().max()) <= 8 * 2.0 ** -20


@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_split_rows_with_infinite_values(d, block):
    """V infinite at one token of a row's last chunk: that column of O is the infinity, the others as without it, for rows
    of two, three and four chunks (the merge takes four at a time)."""
    import paper_2609_34814_amd as W
    mb, n = 41, 41 * block - 7
    g = torch.Generator(device="cuda").manual_seed(d + block)
    q, k, v = (torch.randn(1, 1, n, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = _mask(1, mb, np.random.default_rng(d + block))
    mask[0, 0, 3:7, mb - 1] = 1       # the last block, in the last chunk
    mask = u8_dev(mask)
    plain = W.sparse_attn(q, k, v, mask, block=block)[0, 0]
    v[0, 0, n - 3, 5] = float("inf")
    v[0, 0, n - 2, d - 1] = -float("inf")
    o = W.sparse_attn(q, k, v, mask, block=block)[0, 0]
    for r in (3, 4, 5, 6):
        t = slice(r * block, (r + 1) * block)
        assert bool(torch.isposinf(o[t, 5]).all()) and bool(torch.isneginf(o[t, d - 1]).all()), r
        rest = [c for c in range(d) if c not in (5, d - 1)]
        assert torch.equal(o[t][:, rest], plain[t][:, rest]), r


def test_chunks_of_a_list_with_repeats():
    """A caller-built list that names every block 1,200 times (1.8 M entries, in 1,229 chunks on 256 compute units: entries
    times chunks exceed 2^31): O is that of the plain row, the LSE larger by ln 1200."""
    import paper_2609_34814_amd as W
    mb, d, block, times = 1500, 64, 64, 1200
    n = mb * block
    g = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.randn(1, 1, n, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    vt = W.transpose_v(v, block=block)
    lists = []
    for repeat in (1, times):
        row_ptr = torch.zeros(1, 1, mb + 1, dtype=torch.int32, device="cuda")
        row_ptr[0, 0, 1:] = repeat * mb
        col_idx = torch.zeros(mb * mb, dtype=torch.int32, device="cuda")
        col_idx[:repeat * mb] = torch.arange(mb, dtype=torch.int32, device="cuda").repeat(repeat)
        lists.append((row_ptr, col_idx))
    (o1, l1), (o2, l2) = (W.sparse_attn_vt(q, k, vt, *x, block=block, return_lse=True) for x in lists)
    o1, o2 = o1[0, 0, :block].double(), o2[0, 0, :block].double()
    # float32 sums of 1.2e8 terms, a few thousand per accumulator and chunk: below a bf16 rounding
    assert float((o1 - o2).norm() / o1.norm()) <= 2.0 ** -8
    assert float((l2[0, 0, :block] - l1[0, 0, :block] - np.log(times)).abs().max()) <= 1e-3


def test_slots_outside_the_segments_are_not_computed():
    """A segment table that leaves slots out: their rows keep their old contents, whether they would be split or not."""
    import paper_2609_34814_amd as W
    mb, d, block = 41, 64, 64
    n = mb * block
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(1, 2, n, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = u8_dev(_mask(2, mb, np.random.default_rng(5)))
    want = W.sparse_attn(q, k, v, mask, block=block)
    # head 0 runs slots 3 to 5 alone (slot 6, the full row, is left out); head 1 all
    seg = torch.tensor([[[3, 4, 4, 6, 6], [0, 10, 20, 30, mb]]], dtype=torch.int32, device="cuda")
    run = torch.ones(2, mb, dtype=torch.bool)
    run[0] = False
    for lo, hi in zip(seg[0, 0, :-1].tolist(), seg[0, 0, 1:].tolist()):
        run[0, lo:max(lo, hi)] = True
    out = torch.full_like(want, float("nan"))
    W.sparse_attn(q, k, v, mask, None, seg, block=block, n_xcd=4, out=out)
    for h in range(2):
        for r in range(mb):
            t = slice(r * block, (r + 1) * block)
            if run[h, r]:
                assert torch.equal(out[0, h, t], want[0, h, t]), (h, r)
            else:
                assert bool(torch.isnan(out[0, h, t]).all()), (h, r)


@pytest.mark.parametrize("n_xcd,heads,mb", [(8, 2, 41), (64, 1, 41), (64, 1, 2)])
def test_workspace_without_room_for_split_rows(n_xcd, heads, mb):
    """The sizes that the C calls report: every row whole, within a bf16 rounding of the split rows in a larger one.
    With 64 queues and few rows the task counters lie side by side."""
    import ctypes
    import paper_2609_34814_amd as W
    from paper_2609_34814_amd import _lib as L
    lib, d, block = L.load(), 64, 64
    n = mb * block
    g = torch.Generator(device="cuda").manual_seed(mb)
    q, k, v = (torch.randn(1, heads, n, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = u8_dev(_mask(heads, mb, np.random.default_rng(mb)) if mb > 8 else np.ones((1, heads, mb, mb), np.uint8))
    want = W.sparse_attn(q, k, v, mask, block=block, n_xcd=n_xcd)
    rp, ci = W.compact_mask(mask, seq_len=n, block=block, head_dim=d)
    vt = W.transpose_v(v, block=block)
    shape, size = W.shape_of(1, heads, n, d, block), ctypes.c_size_t(0)
    for call, run in (("wa_attn_workspace_size", lambda **kw: W.sparse_attn(q, k, v, mask, **kw)),
                      ("wa_attn_workspace_size", lambda **kw: W.sparse_attn_csr(q, k, v, rp, ci, **kw)),
                      ("wa_attn_vt_workspace_size", lambda **kw: W.sparse_attn_vt(q, k, vt, rp, ci, **kw))):
        assert getattr(lib, call)(ctypes.byref(shape), ctypes.byref(size)) == 0
        buf = torch.full((size.value + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        out = torch.full_like(want, float("nan"))
        run(block=block, n_xcd=n_xcd, out=out, workspace=buf[:size.value])
        assert bool((buf[size.value:] == 0x5A).all())
        assert float((out.float() - want.float()).norm() / want.float().norm()) <= 2e-4


@pytest.mark.parametrize("d,block,heads,mb,most,few,long,splits", [
    (64, 64, 12, 64, 24, 0, 0, False),      # equal rows, half as many as workgroups: chunks cost more than they save
    (64, 64, 15, 66, 40, 0, 0, False),
    (64, 128, 5, 48, 24, 0, 0, False),
    (128, 128, 5, 48, 40, 0, 0, False),
    (128, 64, 2, 64, 50, 0, 0, True),       # equal rows, few of them
    (64, 128, 2, 48, 40, 0, 0, True),
    (64, 64, 20, 80, 6, 3, 80, True),       # a few long rows
    (128, 128, 12, 100, 8, 4, 100, True),
])
def test_rows_are_split_where_it_pays(d, block, heads, mb, most, few, long, splits):
    """The plan of a call equals the rule, which weighs the longest row against the chunks' cost."""
    rng = np.random.default_rng(mb)
    counts = np.full((heads, mb), most)
    counts.ravel()[rng.permutation(counts.size)[:few]] = long
    chunks, longest, _ = _plan(counts, d, block)
    assert (chunks > 0) == splits
    g = torch.Generator(device="cuda").manual_seed(mb)
    q, k, v = (torch.randn(1, heads, mb * block, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    _, _, got, got_l = _planned(q, k, v, u8_dev(_rows_of(counts, rng)), block)
    assert got == chunks and (not splits or got_l == longest)
