"""GPU parity of the isolated kernels (projection, cache update + attention) against the oracle."""
import numpy as np
import pytest
import torch

import dkv_inputs as D
from dkv_inputs.configs import BF16, FP32
from oracle.attn_update import attn_update as oracle_attn_update
from helpers import rel_err
from gpu_parity import check_close, tolerances
from plans import OWN_LAUNCH, PRODUCT, STAGGER, STREAM_TILES, XCD_GROUP, attn_plan, embed_norm, gather_rows, gemm_plan, launch_head, launch_stream

pytestmark = pytest.mark.gpu


def _dev(x, dtype):
    td = torch.bfloat16 if dtype == BF16 else torch.float32
    return torch.from_numpy(np.ascontiguousarray(x)).to(device="cuda", dtype=td)


@pytest.mark.parametrize("dtype", [BF16, FP32])
@pytest.mark.parametrize("m,n,k", [(1, 128, 64), (2, 384, 4096), (37, 200, 136), (64, 256, 512),
                                   (129, 384, 1024), (300, 130, 72), (513, 256, 256)])
def test_projection_matches_float64_product(dtype, m, n, k):
    import paper_2505_15781_amd as P
    x = D.normal_f32(5, 1, (m, k), bf16=dtype == BF16)
    w = D.normal_f32(5, 2, (n, k), std=0.02, bf16=dtype == BF16)
    y = P.gemm(_dev(x, dtype), _dev(w, dtype), dtype).cpu().numpy()
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    check_close(y, ref, 1e-5, f"gemm {m}x{n}x{k}")


@pytest.mark.parametrize("m", [3, 40, 100])
def test_projection_planned_launch_on_a_weight_matrix_that_is_streamed(m):
    """A weight matrix of 32 MB: with one row of tiles the planner streams it with the non-temporal hint, slices K
    and staggers the K start; the product is the same."""
    import paper_2505_15781_amd as P
    n, k = 4096, 4096
    x = D.normal_f32(7, 1, (m, k), bf16=True)
    w = D.normal_f32(7, 2, (n, k), std=0.02, bf16=True)
    y = P.gemm(_dev(x, BF16), _dev(w, BF16), BF16).cpu().numpy()
    check_close(y, x.astype(np.float64) @ w.astype(np.float64).T, 1e-5, f"gemm {m}x{n}x{k}")


@pytest.mark.parametrize("m,n,k,rule", [
    (150, 24576, 4096, "sliced"), (192, 12288, 4096, ""), (320, 12288, 2048, ""), (384, 24576, 1024, "192 rows"),
    (513, 3584, 4096, "sliced, 192 rows"), (600, 45000, 2048, "grouped, 192 rows"), (1500, 4096, 4096, "grouped"),
    (2048, 4608, 3584, "grouped"), (2049, 4608, 3584, "grouped"), (2049, 512, 4096, "sliced"), (2304, 3584, 18944, "sliced, grouped"),
    (3072, 1024, 8192, "sliced, grouped"), (384, 70000, 2048, "staggered"), (513, 50000, 2048, "staggered, 192 rows")])
def test_projection_planned_launch_from_150_to_3072_rows(m, n, k, rule):
    """Row counts at which the planner takes 192-row tiles, slices K at hundreds to thousands of rows, groups the tiles by XCD,
    and staggers the K start over two or three rows of tiles and several rounds of workgroups; `rule`: what the plan has to
    be for the case to be worth running. fp32 sums of k products of
    N(0, 1) and N(0, 0.02^2): rounding stays below 1e-6 of the largest value, the bar of the other projections is 1e-5."""
    import paper_2505_15781_amd as P
    p = gemm_plan(m, n, k, OWN_LAUNCH)
    rows, workgroups = p.grid(m, n)
    assert (p.split_k > 1) == ("sliced" in rule)
    assert (rows > 1 and p.flags & STAGGER != 0) == ("staggered" in rule)
    assert (p.flags & XCD_GROUP != 0) == ("grouped" in rule)
    assert "192 rows" not in rule or p.tile == "dma_192x256"
    assert "staggered" not in rule or workgroups > 512
    g = torch.Generator(device="cuda").manual_seed(m + n)
    x = torch.randn((m, k), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((n, k), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    y = P.gemm(x, w, BF16).double()
    ref = x.double() @ w.double().T
    assert ((y - ref).norm() / ref.norm()).item() <= 1e-5 and ((y - ref).abs().max() / ref.abs().max()).item() <= 1e-5


@pytest.mark.parametrize("tile", sorted(STREAM_TILES))
@pytest.mark.parametrize("m,n,k,split,rows", [(256, 384, 1024, 1, None), (129, 200, 64, 1, None), (255, 97, 128, 1, 131), (1, 1000, 192, 1, None),
                                              (250, 1000, 2048, 3, None), (193, 96, 704, 2, 64), (256, 3000, 4096, 8, 256)])
def test_projection_of_one_row_of_tiles(tile, m, n, k, split, rows):
    """One to eleven K tiles per slice (fewer than the stages, odd and even against the pairs in which weights are fetched), ragged
    columns, more workgroups than one round, and a device-side row count below the bound: rows past it are not written. Sums
    of k products of N(0, 1) and N(0, 0.02^2), as for the other projection kernels."""
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn((m, k), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((n, k), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    got = launch_stream(x, w, tile, split, None if rows is None else torch.tensor([rows], dtype=torch.int32, device="cuda"))
    live = m if rows is None else rows
    assert torch.isnan(got[:, live:]).all() and not torch.isnan(got[:, :live]).any()
    ref = x[:live].double() @ w.double().T
    err = got[:, :live].double().sum(0) - ref
    assert (err.norm() / ref.norm()).item() <= 1e-5 and (err.abs().max() / ref.abs().max()).item() <= 1e-5


@pytest.mark.parametrize("tile", sorted(STREAM_TILES))
@pytest.mark.parametrize("m,n,k,rows", [(m, n, k, rows) for m, n, k in ((256, 384, 1024), (129, 200, 64), (255, 98, 128), (1, 1000, 192))
                                        for rows in (None, 1, 64, 65, 131) if rows is None or rows <= m])
def test_swiglu_of_one_row_of_tiles(tile, m, n, k, rows):
    """The same sums through the SwiGLU epilogue, with device-side row counts at and across the 64 rows of a multiplying wavefront:
    rows past the count are not written. The result is rounded to bf16: half a unit of 8 significant bits, at most 2^-8 of the
    value; the sums as above."""
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn((m, k), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((n, k), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    y = launch_stream(x, w, tile, 1, None if rows is None else torch.tensor([rows], dtype=torch.int32, device="cuda"), swiglu=True)
    live = m if rows is None else rows
    assert torch.isnan(y[live:]).all() and not torch.isnan(y[:live]).any()
    full = x[:live].double() @ w.double().T
    want = torch.nn.functional.silu(full[:, 0::2]) * full[:, 1::2]
    excess = ((y[:live].double() - want).abs() - 2.0 ** -8 * want.abs()).max() / want.abs().max()
    assert excess.item() <= 1e-5


@pytest.mark.parametrize("kind,split", [("dma_32x128", 1), ("dma_32x128", 3), ("dma_64x128", 2), ("dma_128x128", 1),
                                        ("dma_128x128", 4), ("dma_128x256", 2), ("dma_256x256", 1),
                                        ("dma_256x256", 3), ("dma_128x96", 1), ("dma_128x96", 2),
                                        ("dma_128x192", 1), ("dma_128x192", 3), ("dma_256x192", 1), ("dma_256x192", 2),
                                        ("dma_192x256", 1), ("dma_192x256", 2),
                                        ("reg_64x128", 2)])
@pytest.mark.parametrize("m,n,k", [(1, 128, 64), (37, 200, 192), (129, 384, 1024), (300, 520, 640), (513, 256, 2048)])
def test_every_projection_kernel_on_ragged_shapes(kind, split, m, n, k):
    import paper_2505_15781_amd as P
    if split > max(1, k // 64):
        pytest.skip("more K slices than K tiles")
    x = D.normal_f32(6, 1, (m, k), bf16=True)
    w = D.normal_f32(6, 2, (n, k), std=0.02, bf16=True)
    # the effective number of slices may be smaller than requested; ask the library's own count
    kt = -(-k // 64)
    kps = -(-kt // split)
    split_eff = -(-kt // kps)
    y = P.gemm(_dev(x, BF16), _dev(w, BF16), BF16, kind=kind, split_k=split_eff).cpu().numpy()
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    check_close(y, ref, 1e-5, f"{kind} split {split_eff} {m}x{n}x{k}")


@pytest.mark.parametrize("kind", ["dma_32x128", "dma_64x128", "dma_128x128", "dma_128x256", "dma_256x256",
                                  "dma_128x96", "dma_128x192", "dma_256x192", "dma_192x256"])
@pytest.mark.parametrize("options", [1, 2, 3, 8, 9])
@pytest.mark.parametrize("m,n,k,split", [(5, 128, 256, 1), (129, 384, 1024, 1), (300, 520, 768, 2),
                                         (1100, 1536, 512, 1), (1030, 2048, 640, 2)])
def test_projection_launch_options_leave_the_product_unchanged(kind, options, m, n, k, split):
    """A staggered K loop start and the XCD-grouped tile order only permute work: same product (up to fp32
    summation order); the last two shapes have at least four tile rows, so the grouping is really applied."""
    import paper_2505_15781_amd as P
    x = D.normal_f32(9, 1, (m, k), bf16=True)
    w = D.normal_f32(9, 2, (n, k), std=0.02, bf16=True)
    y = P.gemm(_dev(x, BF16), _dev(w, BF16), BF16, kind=kind, split_k=split, options=options).cpu().numpy()
    check_close(y, x.astype(np.float64) @ w.astype(np.float64).T, 1e-5, f"{kind} options {options} {m}x{n}x{k}")


@pytest.mark.parametrize("kind", ["dma_32x128", "dma_64x128", "dma_128x128", "dma_128x256", "dma_256x256",
                                  "dma_128x96", "dma_128x192", "dma_256x192", "dma_192x256"])
@pytest.mark.parametrize("m,n,k", [(5, 128, 256), (129, 392, 1024), (300, 520, 768)])
def test_projection_with_fused_swiglu_epilogue(kind, m, n, k):
    """Rows of w interleave gate_j, up_j; the epilogue writes silu(gate) * up (the feed-forward's activation)
    as bf16 [m, n/2] instead of the fp32 product. bf16 output: one rounding, 2^-9 relative."""
    import paper_2505_15781_amd as P
    from paper_2505_15781_amd import binding
    x = D.normal_f32(10, 1, (m, k), bf16=True)
    w = D.normal_f32(10, 2, (n, k), std=0.05, bf16=True)
    y = P.gemm(_dev(x, BF16), _dev(w, BF16), BF16, kind=kind, split_k=1,
               options=binding.GEMM_OPT_SWIGLU).float().cpu().numpy()
    prod = x.astype(np.float64) @ w.astype(np.float64).T
    g, u = prod[:, 0::2], prod[:, 1::2]
    check_close(y, g / (1.0 + np.exp(-g)) * u, 4e-3, f"{kind} fused swiglu {m}x{n}x{k}")
    with pytest.raises(P.DkvError) as e:
        P.gemm(_dev(x, BF16), _dev(w, BF16), BF16, kind=kind, split_k=2, options=binding.GEMM_OPT_SWIGLU)
    assert e.value.code == -3


@pytest.mark.parametrize("kind", ["dma_256x256", "dma_256x192", "dma_192x256"])
@pytest.mark.parametrize("k_tiles", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("m,n", [(1, 4), (255, 193), (257, 258), (193, 512)])
def test_eight_wavefront_tiles_at_short_k_and_tile_edges(kind, k_tiles, m, n):
    """The two wavefront groups run one barrier apart and fetch two K tiles ahead: one to five K tiles take every exit
    of that schedule; rows and columns just below and above a tile, widths that are no multiple of 4. fp32 sums of
    64 k_tiles products: 1e-5 is far above their rounding."""
    import paper_2505_15781_amd as P
    k = 64 * k_tiles
    x = D.normal_f32(13, 1, (m, k), bf16=True)
    w = D.normal_f32(13, 2, (n, k), std=0.02, bf16=True)
    y = P.gemm(_dev(x, BF16), _dev(w, BF16), BF16, kind=kind, split_k=1).cpu().numpy()
    check_close(y, x.astype(np.float64) @ w.astype(np.float64).T, 1e-5, f"{kind} {m}x{n}x{k}")


@pytest.mark.parametrize("tile", ["dma_256x256", "dma_256x192", "dma_192x256", "dma_128x192"])
@pytest.mark.parametrize("rows_off,cols_off", [(-1, -1), (1, 1), (0, 0), (-60, 2), (1, 3)])
def test_vocabulary_statistics_of_the_tile_kernels(tile, rows_off, cols_off):
    """Per row and column tile: maximum, sum of exp(x - max), lowest arg max, MASK and columns past the end excluded. Rows and
    columns just below, at and above one tile (and two tiles of columns), widths of every remainder by 4; planted: equal
    maxima in two lanes, two wavefronts and two tiles, MASK as the largest logit, a NaN row, a row past the device's count.
    Maximum and arg max are those of the kernel's own fp32 logits, exactly. The sum adds at most 256 exponentials of |x - max|
    < 64: exp2 of a product rounded to 2^-24 of at most 93 has an error below 93 ln 2 2^-24 = 4e-6, the additions less."""
    import paper_2505_15781_amd as P
    bm, bn = (int(v) for v in tile.split("_")[1].split("x"))
    m, n, k = bm + rows_off, 2 * bn + cols_off, 192
    x, w = D.normal_f32(16, 1, (m, k), std=0.25, bf16=True), D.normal_f32(16, 2, (n, k), std=0.25, bf16=True)
    mask_id = 37
    ties = {3: (5, 6), 7: (17, 90), 20: (2, bn - 1), 33: (bn - 2, bn + 8), 40: (100, 100 + 4)}       # row: equal columns
    for r, (lo, hi) in ties.items():
        w[hi] = w[lo]
        x[r] = 4 * w[lo]
    x[11] = 4 * w[mask_id]
    x[50] = np.nan
    dead = m - 1                                     # not counted by the device: neither read nor written
    x[dead] = np.nan
    xd, wd = _dev(x, BF16), _dev(w, BF16)
    count = torch.tensor([m - 1], dtype=torch.int32, device="cuda")
    logits = torch.zeros((m, n), dtype=torch.float32, device="cuda")
    status = torch.zeros(2, dtype=torch.int32, device="cuda")
    got = launch_head(xd, wd, tile, mask_id, status[:1], count, logits)
    again = launch_head(xd, wd, tile, mask_id, status[:1], count)              # logits not written
    xd[50] = 0
    launch_head(xd, wd, tile, mask_id, status[1:], count)
    assert status.tolist() == [1, 0]
    live = [r for r in range(m - 1) if r != 50]
    assert torch.equal(got[live], again[live])
    lg, got = logits.cpu().numpy(), got.cpu()
    ref = x[live].astype(np.float64) @ w.astype(np.float64).T
    check_close(lg[live], ref, 1e-5, f"{tile} logits {m}x{n}")
    assert (got[dead] == 0x7fc00123).all() and not lg[dead].any()
    mx, sm, ix = got[..., 0].contiguous().view(torch.float32).numpy(), got[..., 1].contiguous().view(torch.float32).numpy(), got[..., 2].numpy()
    for t in range(got.shape[1]):
        cols = np.arange(t * bn, min(n, (t + 1) * bn))
        cols = cols[cols != mask_id]
        part = lg[np.ix_(live, cols)]
        assert np.array_equal(mx[live, t], part.max(axis=1))
        assert np.array_equal(ix[live, t], cols[part.argmax(axis=1)])
        want = np.exp(part.astype(np.float64) - part.max(axis=1, keepdims=True)).sum(axis=1)
        assert np.max(np.abs(sm[live, t] - want) / want) <= 1e-5
    for r, (lo, hi) in ties.items():
        if r in live:
            assert lg[r, lo] == lg[r, hi] == lg[r].max() and ix[r, 0] == lo
    assert lg[11].argmax() == mask_id


@pytest.mark.parametrize("tile", ["dma_32x128", "dma_64x128", "dma_128x128", "dma_128x256", "dma_128x96"])
@pytest.mark.parametrize("rows_off,tiles_n,cols_off,k", [(0, 1, 0, 64), (-1, 1, -90, 128), (1, 2, 1, 192), (-31, 3, -1, 256), (-16, 1, -64, 320)])
def test_vocabulary_statistics_of_four_wavefronts(tile, rows_off, tiles_n, cols_off, k):
    """The reductions over the 32 lanes of a row: columns that end in the first lanes, in the middle and at the end of a tile, every
    logit twice a row (distances over lanes, wavefronts and tiles), a NaN row, one past the device's count; one to five K tiles,
    fewer than are fetched ahead and more. Records against the kernel's own fp32 logits (maximum and arg max exactly, the sum to
    the bound of the test above: no logit is further than 64 from the row's maximum), those against float64."""
    bm, bn = (int(v) for v in tile.split("_")[1].split("x"))
    m, n = max(bm + rows_off, 2), tiles_n * bn + cols_off
    mask_id = n // 3
    g = torch.Generator(device="cuda").manual_seed(m + n)
    x = (torch.randn((m, k), generator=g, device="cuda") * 0.25).to(torch.bfloat16)
    w = (torch.randn((n, k), generator=g, device="cuda") * 0.25).to(torch.bfloat16)
    w[n - n // 2:] = w[:n // 2]
    x[m - 1] = float("nan")
    count = torch.tensor([m - 1], dtype=torch.int32, device="cuda")
    logits, status = torch.zeros((m, n), dtype=torch.float32, device="cuda"), torch.zeros(2, dtype=torch.int32, device="cuda")
    got = launch_head(x, w, tile, mask_id, status[:1], count, logits)
    assert torch.equal(got, launch_head(x, w, tile, mask_id, status[:1], count))        # logits not written
    assert (got[m - 1] == 0x7fc00123).all() and not logits[m - 1].any()
    x[m - 2, k - 1] = float("nan")
    launch_head(x, w, tile, mask_id, status[1:], count)
    assert status.tolist() == [0, 1]
    x[m - 2, k - 1] = 0
    got, lg = launch_head(x, w, tile, mask_id, status[:1], count, logits)[:m - 1], logits[:m - 1]
    ref = x[:m - 1].double() @ w.double().T
    assert ((lg - ref).norm() / ref.norm()).item() <= 1e-5
    lg[:, mask_id] = -float("inf")
    part = torch.nn.functional.pad(lg, (0, -n % bn), value=-float("inf")).view(m - 1, -1, bn)
    top = part.max(dim=2).values
    assert torch.equal(got[..., 0].contiguous().view(torch.float32), top)
    lowest = (part == top[..., None]).int().argmax(dim=2) + bn * torch.arange(part.shape[1], device="cuda")
    assert torch.equal(got[..., 2], lowest.to(torch.int32))
    want = (part.double() - top.double()[..., None]).exp().sum(dim=2)
    assert ((got[..., 1].contiguous().view(torch.float32) - want).abs() / want).max().item() <= 1e-5


@pytest.mark.parametrize("dtype", [BF16, FP32])
@pytest.mark.parametrize("d", [4, 252, 260, 1024, 1028, 2052, 4096, 4100, 8192])
def test_embedded_rows_and_gathered_candidates_in_pieces_of_four(dtype, d):
    """Row lengths around what one, four, eight and 16 wavefronts hold and two pieces a lane, a table that starts one element past
    any alignment, rows past the device's counts. The residual rows and the gathered ones are copies; the norm adds d squares in
    fp32 (lanes, then 64 and 16 of them: at most 28 additions in a row, 2^-24 each, half of it after the root) and rounds three
    products and the reciprocal root: below 2^-19, and with bf16 (seven bits behind the leading one) half a unit of 2^-7 more."""
    rows, L, V = 7, 11, 13
    t = torch.bfloat16 if dtype == BF16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(d)
    table = torch.randn(V * d + 1, generator=g, device="cuda").to(t)[1:].view(V, d)
    gain = (torch.rand(d + 1, generator=g, device="cuda") + 0.5)[1:]
    tokens = torch.randint(V, (2, L), generator=g, device="cuda", dtype=torch.int32)
    pos, seq = (torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([0, 3, 10, 1, 2, 9, 0], [0, 0, 0, 1, 1, 1, 1]))
    counts = torch.tensor([rows - 1, 3], dtype=torch.int32, device="cuda")
    h, a = torch.zeros((rows, d), device="cuda"), torch.zeros((rows, d), dtype=t, device="cuda")
    stamp = torch.zeros((2, L), dtype=torch.int32, device="cuda")
    embed_norm(table, tokens, pos, seq, counts, gain, h, a, stamp, 1e-5, 5)
    live = slice(0, rows - 1)
    ids = tokens[seq[live].long(), pos[live].long()].long()
    want = table[ids].double()
    assert torch.equal(h[live].double(), want) and not h[rows - 1].any() and not a[rows - 1].any()
    assert stamp.count_nonzero().item() == rows - 1 and (stamp[seq[live].long(), pos[live].long()] == 5).all()
    want = want / (want.square().mean(dim=1, keepdim=True) + 1e-5).sqrt() * gain.double()
    bound = 2.0 ** -19 + (2.0 ** -8 if dtype == BF16 else 0.0)
    assert ((a[live].double() - want).abs() <= bound * want.abs()).all()
    picked = torch.zeros((4, d), dtype=t, device="cuda")
    gather_rows(a, torch.tensor([5, 0, 5, 2], dtype=torch.int32, device="cuda"), counts, picked)
    assert torch.equal(picked[:3], a[[5, 0, 5]]) and not picked[3].any()


@pytest.mark.parametrize("d", [4, 60, 128, 252, 256, 260, 512, 1024, 1028, 2048, 4096])
def test_embedded_rows_in_fp32_keep_the_order_of_their_sums(d):
    """Two candidates of a step can be equal but for a rounding, so another order of the sums would commit the other one: bit for
    bit, a lane's four squares (fused as the compiler contracts them; in float64 a product is exact), the 64 lanes by partners 32,
    16 ... 1 apart, the wavefronts in ascending order, and the reciprocal root, division and products as IEEE rounds them."""
    rows, V = 5, 9
    g = torch.Generator(device="cuda").manual_seed(d)
    table, gain = torch.randn((V, d), generator=g, device="cuda"), torch.rand(d, generator=g, device="cuda") + 0.5
    tokens = torch.arange(rows, device="cuda", dtype=torch.int32)[None].contiguous()
    zero = torch.zeros(rows, dtype=torch.int32, device="cuda")
    h, a = torch.zeros((rows, d), device="cuda"), torch.zeros((rows, d), device="cuda")
    embed_norm(table, tokens, tokens[0], zero, torch.tensor([rows, 0], dtype=torch.int32, device="cuda"), gain, h, a, torch.zeros_like(tokens), 1e-5, 1)
    x = table[:rows].cpu().numpy()
    v = np.zeros((rows, -(-d // 256) * 256), np.float32)
    v[:, :d] = x
    v = v.reshape(rows, -1, 64, 4)
    part = v[..., 0] * v[..., 0]
    for e in (1, 2, 3):
        part = (v[..., e].astype(np.float64) ** 2 + part).astype(np.float32)
    for apart in (32, 16, 8, 4, 2, 1):
        part = part + part[:, :, np.arange(64) ^ apart]
    total = np.zeros(rows, np.float32)
    for wavefront in range(part.shape[1]):
        total = total + part[:, wavefront, 0]
    root = np.float32(1) / np.sqrt(total / np.float32(d) + np.float32(1e-5))
    want = x * root[:, None] * gain.cpu().numpy()
    assert (h.cpu().numpy() == x).all() and (a.cpu().numpy() == want).all()


@pytest.mark.parametrize("m,n,k", [(1, 2, 4), (16, 16, 64), (17, 30, 60), (64, 130, 68), (65, 16, 1028), (128, 4096, 64),
                                   (129, 4096, 64), (16, 16, 128), (20, 20, 132)])
def test_fp32_projection_of_few_rows_at_tile_edges(m, n, k):
    """16x16 tiles, K in pieces of 128: row, column and K remainders, and the two sides of the line beyond which 64x64
    tiles take over. fp32 sums of at most 1028 products."""
    import paper_2505_15781_amd as P
    x = D.normal_f32(14, 1, (m, k))
    w = D.normal_f32(14, 2, (n, k), std=0.02)
    y = P.gemm(_dev(x, FP32), _dev(w, FP32), FP32).cpu().numpy()
    check_close(y, x.astype(np.float64) @ w.astype(np.float64).T, 1e-5, f"fp32 gemm {m}x{n}x{k}")


def test_projection_rejects_unknown_option_bits():
    import paper_2505_15781_amd as P
    x = _dev(D.normal_f32(6, 1, (4, 64), bf16=True), BF16)
    w = _dev(D.normal_f32(6, 2, (8, 64), bf16=True), BF16)
    with pytest.raises(P.DkvError) as e:
        P.gemm(x, w, BF16, kind="dma_32x128", split_k=1, options=16)
    assert e.value.code == -1


@pytest.mark.parametrize("kind", ["dma_32x128", "dma_64x128", "dma_128x128", "dma_128x256", "dma_256x256"])
@pytest.mark.parametrize("m,n,k", [(5, 128, 256), (37, 200, 512), (129, 384, 1024), (300, 520, 768), (257, 1536, 4096)])
def test_three_quarter_k_share_covers_every_tile_twice(kind, m, n, k):
    """Workgroups that take 3/4 of a tile's K range each (possibly ending one tile and starting the next)."""
    import paper_2505_15781_amd as P
    x = D.normal_f32(8, 1, (m, k), bf16=True)
    w = D.normal_f32(8, 2, (n, k), std=0.02, bf16=True)
    y = P.gemm(_dev(x, BF16), _dev(w, BF16), BF16, kind=kind, split_k=-1).cpu().numpy()
    check_close(y, x.astype(np.float64) @ w.astype(np.float64).T, 1e-5, f"{kind} 3/4 share {m}x{n}x{k}")


def test_projection_kernel_rejects_shapes_it_cannot_take():
    import paper_2505_15781_amd as P
    x = _dev(D.normal_f32(6, 1, (4, 72), bf16=True), BF16)
    w = _dev(D.normal_f32(6, 2, (8, 72), bf16=True), BF16)
    with pytest.raises(P.DkvError) as e:
        P.gemm(x, w, BF16, kind="dma_128x128", split_k=1)      # K = 72 is not a multiple of 64
    assert e.value.code == -3
    y = P.gemm(x, w, BF16, kind="reg_64x128", split_k=1).cpu().numpy()
    check_close(y, x.float().cpu().numpy().astype(np.float64) @ w.float().cpu().numpy().astype(np.float64).T, 1e-5, "reg")


def _attn_case(shape, n_active, seed, ragged=None, q_scale=1.0, kernel=None):
    """`kernel`: the route that the case is there for (a changed dispatch must not leave a kernel without its tests), with the
    number of key slices behind a slash where that counts."""
    import paper_2505_15781_amd as P
    if kernel:
        p = attn_plan(shape, n_active if ragged is None else max(ragged))
        assert (f"{p.kernel}/{p.splits}" if "/" in kernel else p.kernel) == kernel
    c = D.attn_update_case(shape, n_active, seed, ragged=ragged)
    c["q"] = c["q"] * np.float32(q_scale)            # a power of two: still exact bfloat16 values
    dt = shape.dtype
    kc, vc = _dev(c["k_cache"], dt), _dev(c["v_cache"], dt)
    rows = int(c["active_off"][-1])
    max_rows = int(np.max(np.diff(c["active_off"]))) if shape.batch else 0
    q, kn, vn = _dev(c["q"], dt), _dev(c["k_new"], dt), _dev(c["v_new"], dt)
    idx = torch.from_numpy(c["active_idx"]).cuda()
    off = torch.from_numpy(c["active_off"]).cuda()
    out = torch.zeros((max(rows, 1), shape.n_q_heads, shape.head_dim), dtype=q.dtype, device="cuda")
    nb = P.attn_update_workspace_bytes(shape.batch, shape.n_q_heads, shape.n_kv_heads, shape.seq_len,
                                       shape.head_dim, dt, max_rows)
    ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
    P.attn_update(kc, vc, q, kn, vn, idx, off, out, rows, max_rows, dt, ws)
    torch.cuda.synchronize()
    rk, rv = c["k_cache"].astype(np.float64), c["v_cache"].astype(np.float64)
    ref = oracle_attn_update(rk, rv, c["q"], c["k_new"], c["v_new"], c["active_idx"], c["active_off"])
    # the scatter is a copy: cache contents must be bit-exact
    assert np.array_equal(kc.float().cpu().numpy().astype(np.float64), rk)
    assert np.array_equal(vc.float().cpu().numpy().astype(np.float64), rv)
    if rows:
        check_close(out[:rows].float().cpu().numpy(), ref, tolerances(dt), f"attention A={n_active} {ragged}")


@pytest.mark.parametrize("dh", [128, 64])
def test_attention_small_ragged_gqa_bf16(dh):
    shape = D.AttnUpdateShape(batch=3, n_q_heads=6, n_kv_heads=2, seq_len=203, head_dim=dh, dtype=BF16)
    _attn_case(shape, None, 31, ragged=[5, 0, 37])
    _attn_case(shape, None, 32, ragged=[1, 1, 1])
    _attn_case(shape, None, 33, ragged=[203, 64, 17])


@pytest.mark.parametrize("dh", [128, 64])
def test_attention_key_slices_across_workgroups(dh):
    """Few (sequence, head) pairs and many keys: the keys are sliced over several workgroups and merged by
    the second kernel; 2085 keys leave a ragged last tile and an uneven deal of tiles to the wavefronts."""
    shape = D.AttnUpdateShape(batch=1, n_q_heads=4, n_kv_heads=2, seq_len=2085, head_dim=dh, dtype=BF16)
    _attn_case(shape, None, 34, ragged=[21])
    shape = D.AttnUpdateShape(batch=2, n_q_heads=2, n_kv_heads=2, seq_len=1031, head_dim=dh, dtype=BF16)
    _attn_case(shape, None, 35, ragged=[3, 40])


@pytest.mark.parametrize("batch,q_heads,kv_heads,seq_len,dh,ragged,kernel", [
    (2, 20, 4, 1301, 128, [20, 11], "ksplit1x8/4"), (8, 4, 4, 1301, 128, [20, 0, 1, 17, 16, 20, 0, 5], "ksplit1x8/3"),      # 7 and 2 groups
    (1, 32, 32, 737, 128, [5], "ksplit1x8/3"), (2, 32, 32, 769, 128, [3, 0], "ksplit1x8/3"),                               # 4 and 8 pairs per XCD
    (1, 28, 4, 1100, 128, [33], "ksplit1x8/2"), (1, 4, 4, 6000, 128, [20], "ksplit1x8/8"), (1, 2, 2, 16500, 128, [3], "ksplit1x8/13"),
    (4, 28, 4, 2053, 128, [17, 0, 3, 9], "ksplit2x8/4"), (1, 2, 2, 4500, 128, [200], "ksplit2x8/4"),                        # two tiles per item
    (3, 12, 12, 3073, 128, [64, 0, 33], "ksplit2x8/3"),
    (1, 4, 1, 4008, 128, [131], "ksplit2x8/3"), (1, 7, 1, 7026, 128, [153], "ksplit2x8/3"), (1, 8, 1, 7514, 64, [65], "ksplit2x8/3"),   # 2, 4, 2 rounds
    (1, 2, 2, 1543, 64, [9], "ksplit1x8/3"), (4, 28, 4, 2053, 64, [17, 0, 3, 9], "ksplit1x8/2"), (2, 4, 2, 6001, 64, [33, 5], "ksplit1x8/6"),
    (1, 2, 2, 4500, 64, [200], "ksplit2x8/4"),
    (21, 8, 8, 200, 128, [40, 33, 0] * 7, "ksplit1x4/1"), (21, 8, 8, 200, 64, [40, 33, 0] * 7, "ksplit1x4/1")])
def test_attention_key_slices_of_every_number(batch, q_heads, kv_heads, seq_len, dh, ragged, kernel):
    """Two to 13 slices of the keys, of one- and two-tile items, with several query groups and with one, the cache update fused (64
    rows and fewer) and not, sequences without rows; ragged last tiles and slices of unequal length; workgroups in several rounds."""
    _attn_case(D.AttnUpdateShape(batch, q_heads, kv_heads, seq_len, dh, dtype=BF16), None, 66, ragged=ragged, kernel=kernel)


def test_attention_many_query_tiles_per_head():
    """Several blocks of 128 query rows per kv head (GQA group of 8 and 79 rows: 5 blocks, almost all full), and a count
    that leaves the last block almost empty (66 rows: 16 of its 128 query rows)."""
    shape = D.AttnUpdateShape(batch=16, n_q_heads=128, n_kv_heads=16, seq_len=300, head_dim=128, dtype=BF16)
    _attn_case(shape, 79, 36, kernel="wide")
    _attn_case(shape, 66, 37, kernel="wide")


@pytest.mark.parametrize("seq_len", [64, 100, 192, 300, 512])
def test_attention_wide_blocks_over_one_to_eight_key_tiles(seq_len):
    """Several blocks of query rows per pair (4 x 16 kv heads x 4 or 5 blocks): key counts of 1, 2 (ragged), 3, 5 (ragged)
    and 8 tiles, i.e. odd and even numbers of the tiles that alternate between the two LDS stages; 66 rows leave the last
    block almost empty."""
    shape = D.AttnUpdateShape(batch=4, n_q_heads=128, n_kv_heads=16, seq_len=seq_len, head_dim=128, dtype=BF16)
    n = min(79, seq_len)
    _attn_case(shape, n, 44, kernel="wide")
    _attn_case(shape, min(66, seq_len), 45, kernel="wide")


def test_attention_wide_blocks_with_ragged_sequences():
    """Sequences with no active row at all, with every position active (first and last included) and with a few: one block
    of query rows per (sequence, kv head), and several."""
    shape = D.AttnUpdateShape(batch=4, n_q_heads=64, n_kv_heads=64, seq_len=300, head_dim=128, dtype=BF16)
    _attn_case(shape, None, 52, ragged=[100, 0, 128, 5], kernel="wide")
    shape = D.AttnUpdateShape(batch=4, n_q_heads=128, n_kv_heads=16, seq_len=300, head_dim=128, dtype=BF16)
    _attn_case(shape, None, 53, ragged=[79, 0, 300, 5], kernel="wide")


@pytest.mark.parametrize("batch,heads,kv_heads,seq_len,ragged,grid", [
    (7, 24, 6, 170, [0, 33, 170, 0, 64, 1, 0], 288), (7, 35, 5, 200, [128, 0, 0, 7, 200, 0, 19], 440),
    (15, 32, 32, 130, [0, 128, 3, 0, 127, 65, 0, 1] + [128, 0, 2, 64, 0, 5, 90], 480), (6, 32, 32, 260, [260, 0, 129, 128, 1, 257], 0)])
def test_attention_wide_blocks_with_rows_come_first(batch, heads, kv_heads, seq_len, ragged, grid):
    """Launches of 257 to 511 workgroups hand out the blocks that hold query rows before the others, counted per XCD over its
    (sequence, kv head) pairs: pairs that are no multiple of 8 (42 and 35), sequences without rows first, in between and
    last, exactly full blocks, 60 pairs on an XCD; and a launch beyond (576), which keeps the plain order."""
    shape = D.AttnUpdateShape(batch=batch, n_q_heads=heads, n_kv_heads=kv_heads, seq_len=seq_len, head_dim=128, dtype=BF16)
    p = attn_plan(shape, max(ragged))
    workgroups = -(-batch * kv_heads // 8) * 8 * p.q_blocks
    assert workgroups == grid or (grid == 0 and workgroups >= 512)
    _attn_case(shape, None, 61, ragged=ragged, kernel="wide")


@pytest.mark.parametrize("seq_len,rows", [(16, 16), (17, 17), (32, 20), (33, 33), (63, 15), (65, 65), (97, 16), (129, 31), (160, 100)])
def test_attention_wide_query_blocks_at_tile_edges(seq_len, rows):
    """Blocks of 128 query rows, 32 per wavefront (12 x 16 kv heads of 8 query heads): one to three key tiles of 64, a
    half tile of 32 keys that is full, ragged or masked as a whole, query rows that fill the last block or leave one
    active row (8 query rows) in it."""
    shape = D.AttnUpdateShape(batch=12, n_q_heads=128, n_kv_heads=16, seq_len=seq_len, head_dim=128, dtype=BF16)
    _attn_case(shape, rows, 54, kernel="wide")


@pytest.mark.parametrize("seq_len", [768, 769, 832, 833, 900])
def test_attention_one_query_block_over_long_sequences(seq_len):
    """One block of query rows per (sequence, kv head) and at least 12 key tiles: the kernels that share K/V tiles between 8
    wavefronts (fewer than 512 pairs, two tiles on their way) and 4 (from 512 on). Full and ragged last tiles, 12 to 15
    tiles: both exits of the two-tile loop; sequences without active rows, with a full block, and, in the grouped form,
    with query rows of one active row in several heads."""
    shape = D.AttnUpdateShape(batch=4, n_q_heads=64, n_kv_heads=64, seq_len=seq_len, head_dim=128, dtype=BF16)
    _attn_case(shape, None, 55, ragged=[100, 0, 128, 5], kernel="shared8")
    shape = D.AttnUpdateShape(batch=16, n_q_heads=32, n_kv_heads=32, seq_len=seq_len, head_dim=128, dtype=BF16)
    _attn_case(shape, None, 57, ragged=[100, 0, 128, 5] + [65, 127, 1, 33] * 3, kernel="shared4")
    shape = D.AttnUpdateShape(batch=32, n_q_heads=64, n_kv_heads=16, seq_len=seq_len, head_dim=128, dtype=BF16)
    _attn_case(shape, None, 58, ragged=[17, 0, 32, 5] * 8, kernel="shared4")


@pytest.mark.parametrize("dh", [128, 64])
def test_attention_many_small_items(dh):
    """More (sequence, head, query group) items than compute units: the key-split kernel in its
    4-wavefront form, two workgroups per compute unit, with the cache update fused (40 rows per sequence)."""
    shape = D.AttnUpdateShape(batch=20, n_q_heads=16, n_kv_heads=16, seq_len=150, head_dim=dh, dtype=BF16)
    _attn_case(shape, 40, 38)


@pytest.mark.parametrize("q_scale", [16.0, 0.0])
def test_attention_peaked_and_flat_softmax(q_scale):
    """Scores with a standard deviation of 16 (after the 1/sqrt(d_h)): almost one-hot probabilities, running maxima
    that keep rising over the key tiles and rescale the output; and all-zero queries: every key weighs the same, the
    output is the mean of V. Through every kernel: key-split with 8 and 4 wavefronts and one and two query tiles per item, sliced and
    not, wide query blocks, both forms of the shared tiles, generic."""
    for shape, n, seed, ragged, kernel in [
            (D.AttnUpdateShape(batch=2, n_q_heads=4, n_kv_heads=2, seq_len=1031, head_dim=128, dtype=BF16), None, 46, [3, 40], "ksplit1x8/3"),
            (D.AttnUpdateShape(batch=4, n_q_heads=8, n_kv_heads=4, seq_len=2053, head_dim=128, dtype=BF16), None, 62, [45, 0, 3, 17], "ksplit2x8/4"),
            (D.AttnUpdateShape(batch=4, n_q_heads=32, n_kv_heads=32, seq_len=300, head_dim=128, dtype=BF16), None, 63, [3, 40, 0, 33], "ksplit2x8/1"),
            (D.AttnUpdateShape(batch=5, n_q_heads=16, n_kv_heads=16, seq_len=150, head_dim=128, dtype=BF16), None, 64, [3, 40, 0, 33, 16], "ksplit1x8/1"),
            (D.AttnUpdateShape(batch=21, n_q_heads=8, n_kv_heads=8, seq_len=150, head_dim=128, dtype=BF16), 40, 65, None, "ksplit1x4"),
            (D.AttnUpdateShape(batch=20, n_q_heads=16, n_kv_heads=16, seq_len=150, head_dim=128, dtype=BF16), 40, 50, None, "ksplit2x4"),
            (D.AttnUpdateShape(batch=4, n_q_heads=128, n_kv_heads=16, seq_len=300, head_dim=128, dtype=BF16), 79, 47, None, "wide"),
            (D.AttnUpdateShape(batch=16, n_q_heads=128, n_kv_heads=16, seq_len=200, head_dim=128, dtype=BF16), 66, 48, None, "wide"),
            (D.AttnUpdateShape(batch=4, n_q_heads=64, n_kv_heads=64, seq_len=833, head_dim=128, dtype=BF16), None, 59, [100, 0, 128, 5], "shared8"),
            (D.AttnUpdateShape(batch=16, n_q_heads=32, n_kv_heads=32, seq_len=833, head_dim=128, dtype=BF16), None, 60,
             [128, 0, 70, 5] + [65, 127, 1, 33] * 3, "shared4"),
            (D.AttnUpdateShape(batch=2, n_q_heads=4, n_kv_heads=4, seq_len=70, head_dim=32, dtype=FP32), None, 49, [9, 33], "generic")]:
        _attn_case(shape, n, seed, ragged=ragged, q_scale=q_scale, kernel=kernel)


def test_attention_generic_paths():
    _attn_case(D.AttnUpdateShape(batch=2, n_q_heads=4, n_kv_heads=4, seq_len=70, head_dim=32, dtype=FP32),
               None, 41, ragged=[9, 33])
    _attn_case(D.AttnUpdateShape(batch=2, n_q_heads=4, n_kv_heads=2, seq_len=70, head_dim=32, dtype=BF16),
               None, 42, ragged=[9, 33])
    _attn_case(D.AttnUpdateShape(batch=1, n_q_heads=2, n_kv_heads=1, seq_len=40, head_dim=128, dtype=FP32),
               None, 43, ragged=[7])


def _shifted(t):
    """A copy of t that starts one element behind a 16-byte boundary."""
    buf = torch.empty(t.numel() + 17, dtype=t.dtype, device=t.device)
    lead = (-buf.data_ptr() % 16) // t.element_size() + 1
    view = buf[lead:lead + t.numel()].view(t.shape)
    assert view.data_ptr() % 16 == t.element_size()
    return view.copy_(t)


@pytest.mark.parametrize("dtype,dh", [(FP32, 32), (FP32, 128), (BF16, 32)])
def test_generic_attention_takes_arrays_at_any_element_boundary(dtype, dh):
    """Where the header asks for no alignment, four-element loads and stores may start at any element: bit-identical."""
    import paper_2505_15781_amd as P
    B, Hq, Hkv, L, A = 2, 4, 2, 70, 9
    c = D.attn_update_case(D.AttnUpdateShape(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=L, head_dim=dh, dtype=dtype), A, 56)
    idx, off = torch.from_numpy(c["active_idx"]).cuda(), torch.from_numpy(c["active_off"]).cuda()
    got = []
    for place in (lambda t: t, _shifted):
        # the cache update moves whole 16-byte pieces: the cache and the new rows stay on their boundaries
        kc, vc, kn, vn = (_dev(c[n], dtype) for n in ("k_cache", "v_cache", "k_new", "v_new"))
        q = place(_dev(c["q"], dtype))
        out = place(torch.zeros_like(q))
        P.attn_update(kc, vc, q, kn, vn, idx, off, out, B * A, A, dtype, None)
        got.append(out.clone())
    torch.cuda.synchronize()
    assert torch.equal(*got)


@pytest.mark.parametrize("dtype,kind,m,n,k,options", [(FP32, "simt", 20, 24, 132, 0), (BF16, "dma_256x256", 40, 72, 128, 0),
                                                      (BF16, "dma_192x256", 40, 72, 128, 0), (BF16, "dma_256x192", 40, 80, 128, 4)])
def test_projection_writes_results_at_any_element_boundary(dtype, kind, m, n, k, options):
    """fp32 product, fp32 operands and the bf16 result of the fused SwiGLU one element behind a 16-byte boundary."""
    import paper_2505_15781_amd as P
    from paper_2505_15781_amd import binding as b
    x, w = _dev(D.normal_f32(15, 1, (m, k), bf16=True), dtype), _dev(D.normal_f32(15, 2, (n, k), bf16=True), dtype)
    y = P.gemm(x, w, dtype, kind=kind, split_k=1, options=options)
    ys = _shifted(torch.zeros_like(y))
    if dtype == FP32:                       # bf16 operands travel in 16-byte pieces
        x, w = _shifted(x), _shifted(w)
    b._check(b.lib.dkv_gemm_with(b._ptr(x), b._ptr(w), b._ptr(ys), m, n, k, dtype, b.GEMM_KINDS[kind], 1, options, None, 0, b._stream()))
    torch.cuda.synchronize()
    assert torch.equal(y, ys)


@pytest.mark.parametrize("dtype,dh,seq_len,bits", [
    (FP32, 32, 70, "27f06425927224fcafa23fd4605d4719676c91d7"),
    (FP32, 32, 1300, "b8d71dbcf465e04db1147b46de1d5486de8bc196"),
    (FP32, 64, 64, "8130a4842fe545111c01d83211251a7cee0988e7"),
    (FP32, 64, 1300, "104d3c3b317fe1e15631335c5e67f7972f10d35e"),
    (FP32, 128, 64, "efed2095d0de6a39965b4edbfca5487e638c6c11"),
    (FP32, 128, 517, "809ec4c9b3fd6be1aec076ee1aa3038aa9d830a4"),
    (BF16, 32, 200, "b025b4d48950a493e2bcf393f768665cf67e162d")])
def test_generic_attention_keeps_the_order_of_its_sums(dtype, dh, seq_len, bits):
    """Two candidates of a step can be equal but for a rounding, so another order of the sums, or another choice of which
    product is rounded before it is added, would commit the other one: the results are held to the bits that one output
    vector per lane and a butterfly over the lanes gave (SHA-1 of the output array), over one chunk of 64 keys and many, whole
    and cut."""
    import hashlib
    import paper_2505_15781_amd as P
    B, Hq, Hkv, A = 2, 4, 2, 31
    c = D.attn_update_case(D.AttnUpdateShape(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=seq_len, head_dim=dh, dtype=dtype), A, 64)
    kc, vc, kn, vn, q = (_dev(c[n], dtype) for n in ("k_cache", "v_cache", "k_new", "v_new", "q"))
    out = torch.zeros_like(q)
    P.attn_update(kc, vc, q, kn, vn, torch.from_numpy(c["active_idx"]).cuda(), torch.from_numpy(c["active_off"]).cuda(), out, B * A, A,
                  dtype, None)
    got = hashlib.sha1(out.view(torch.int16 if dtype == BF16 else torch.int32).cpu().numpy().tobytes()).hexdigest()
    assert got == bits


def test_attention_no_rows_is_a_no_op():
    shape = D.AttnUpdateShape(batch=2, n_q_heads=4, n_kv_heads=2, seq_len=64, head_dim=128, dtype=BF16)
    _attn_case(shape, 0, 51)


@pytest.mark.parametrize("n_active", D.CONFIG1_ACTIVE_SIZES)
def test_attention_microbenchmark_configuration_full_size(n_active):
    _attn_case(D.CONFIG1_SHAPE, n_active, 1100 + D.CONFIG1_ACTIVE_SIZES.index(n_active))


@pytest.mark.parametrize("dtype", [BF16, FP32])
def test_concat_reorder_operator_reproduces_the_compact_layout(dtype):
    """The paper's cache operator (Appendix A) on its compact layout, bit for bit: cached rows left, new rows
    right, gathered into the next step's order given by the oracle's index bookkeeping (which the worked
    example of the appendix pins)."""
    import paper_2505_15781_amd as P
    from oracle import schedule as S
    B, H, L, dh = 3, 2, 23, 64
    rng = np.random.default_rng(5)
    full_k = D.normal_f32(12, 1, (B, H, L, dh), bf16=dtype == BF16)      # K/V of every position, position order
    full_v = D.normal_f32(12, 2, (B, H, L, dh), bf16=dtype == BF16)
    n_c = 9
    kc, vc, kn, vn, take, want_k, want_v = [], [], [], [], [], [], []
    for b in range(B):
        unm_prev = sorted(rng.choice(L, size=n_c, replace=False).tolist())            # cached at this step
        rest = [p for p in range(L) if p not in unm_prev]
        unm_next = sorted(unm_prev + rng.choice(rest, size=2, replace=False).tolist())   # two more next step
        layout_prev, layout_next, mapping, _ = S.reorder_map(unm_prev, unm_next, L)
        kc.append(full_k[b][:, layout_prev[:n_c]]); vc.append(full_v[b][:, layout_prev[:n_c]])
        kn.append(full_k[b][:, layout_prev[n_c:]]); vn.append(full_v[b][:, layout_prev[n_c:]])
        take.append(mapping)
        want_k.append(full_k[b][:, layout_next]); want_v.append(full_v[b][:, layout_next])
    dev = lambda xs: _dev(np.stack(xs), dtype)
    tk = torch.tensor(np.asarray(take, dtype=np.int32), device="cuda")
    ko, vo = P.concat_reorder(dev(kc), dev(vc), dev(kn), dev(vn), tk, dtype)
    assert np.array_equal(ko.float().cpu().numpy(), np.stack(want_k))
    assert np.array_equal(vo.float().cpu().numpy(), np.stack(want_v))


def test_bad_arguments_are_errors_not_faults():
    import paper_2505_15781_amd as P
    shape = D.AttnUpdateShape(batch=1, n_q_heads=2, n_kv_heads=1, seq_len=40, head_dim=48, dtype=BF16)
    kc = torch.zeros((1, 1, 40, 48), dtype=torch.bfloat16, device="cuda")
    q = torch.zeros((1, 2, 48), dtype=torch.bfloat16, device="cuda")
    kn = torch.zeros((1, 1, 48), dtype=torch.bfloat16, device="cuda")
    idx = torch.zeros(1, dtype=torch.int32, device="cuda")
    off = torch.tensor([0, 1], dtype=torch.int32, device="cuda")
    with pytest.raises(P.DkvError) as e:
        P.attn_update(kc, kc.clone(), q, kn, kn, idx, off, q.clone(), 1, 1, BF16, None)
    assert e.value.code == -3 and "head_dim" in str(e.value)


def test_yardstick_kernels_copy_exactly_and_report_their_flops():
    """The benchmark's yardsticks: the copy kernel moves every byte (it calibrates the HBM byte counters), the MFMA loop
    reports the flops of its launch, and the three measured rates are of the chip's order of magnitude."""
    import ctypes as C
    from paper_2505_15781_amd import binding as b
    n = (1 << 20) + 48
    src = torch.randint(0, 255, (n,), dtype=torch.uint8, device="cuda")
    dst = torch.zeros_like(src)
    b._check(b.lib.dkv_peak_copy(b._ptr(src), b._ptr(dst), n, b._stream()))
    torch.cuda.synchronize()
    assert torch.equal(src, dst)
    assert b.lib.dkv_peak_copy(b._ptr(src), b._ptr(dst), n - 1, b._stream()) == -1      # not a multiple of 16 bytes
    sink = torch.zeros(1 << 21, dtype=torch.uint8, device="cuda")
    flops = C.c_double(0.0)
    b._check(b.lib.dkv_peak_mfma(b._ptr(sink), 10, C.byref(flops), b._stream()))
    torch.cuda.synchronize()
    assert flops.value == 2048 * 4 * 10 * 4 * 2.0 * 32 * 32 * 16 and not sink.any()
    p = b.measured_peaks(reps=2)
    assert 1000 < p["hbm_read_GBps"] < 8000 and 1000 < p["hbm_copy_GBps"] < 8000 and 300 < p["mfma_bf16_TFLOPs"] < 2600


def test_profile_report_counts_the_bytes_each_projection_really_moves():
    """dkv_profile_begin / end: per kernel kind launches and algorithmic bytes and flops; gate/up with the fused
    SwiGLU counts its bf16 [M, N/2] output, the vocabulary projection none (its epilogue keeps statistics only)."""
    import paper_2505_15781_amd as P
    from paper_2505_15781_amd import binding
    from dkv_inputs.configs import ModelShape, RunShape
    m = ModelShape(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ffn=384, vocab=520, mask_id=519,
                   dtype=BF16)
    r = RunShape(batch=2, prompt_len=8, gen_len=8, steps=8, block_len=8, refresh_interval=4)
    g = P.DkvRun(m, r, binding.random_weights(m, 3), D.prompt_tokens(m, r, 4))
    g.profile_begin()
    g.denoise_step(0)
    prof = g.profile_end()
    rows, cands, d, F, V = 2 * 16, 2 * 8, m.d_model, m.d_ffn, m.vocab
    nqkv, qn = m.qkv_rows, m.n_q_heads * m.head_dim
    proj = lambda M, N, K, out: (M * K + N * K) * 2 + out
    want_bytes = m.n_layers * (proj(rows, nqkv, d, 4 * rows * nqkv) + proj(rows, d, qn, 4 * rows * d) +
                               proj(rows, 2 * F, d, 2 * rows * F) + proj(rows, d, F, 4 * rows * d)) + proj(cands, V, d, 0)
    want_flops = m.n_layers * 2.0 * rows * d * (nqkv + qn + 2 * F + F) + 2.0 * cands * V * d
    got = [v for k, v in prof.items() if k != "attention" and v["launches"]]
    assert sum(v["launches"] for v in got) == 4 * m.n_layers + 1
    assert sum(v["bytes"] for v in got) == want_bytes and sum(v["flops"] for v in got) == want_flops
    assert prof["attention"]["launches"] == m.n_layers
    g.close()


def test_profile_report_keeps_the_projection_kernels_apart():
    """A step whose Q/K/V projection runs on the 256-row tiles and whose down projection has a K that is no multiple of 64: each
    kernel in a place of its own."""
    import paper_2505_15781_amd as P
    from paper_2505_15781_amd import binding
    from dkv_inputs.configs import ModelShape, RunShape
    m = ModelShape(n_layers=1, d_model=4096, n_q_heads=36, n_kv_heads=9, head_dim=128, d_ffn=200, vocab=520, mask_id=519, dtype=BF16)
    r = RunShape(batch=1, prompt_len=128, gen_len=32, steps=32, block_len=32, refresh_interval=4)
    rows, d, qkv = 160, m.d_model, m.qkv_rows
    assert gemm_plan(rows, qkv, d, PRODUCT).kind in STREAM_TILES.values() and gemm_plan(rows, d, m.d_ffn, PRODUCT).tile == "reg_64x128"
    streams = [(n, k) for n, k in ((qkv, d), (d, 36 * 128)) if gemm_plan(rows, n, k, PRODUCT).kind in STREAM_TILES.values()]
    g = P.DkvRun(m, r, binding.random_weights(m, 3), D.prompt_tokens(m, r, 4))
    g.profile_begin()
    g.denoise_step(0)
    prof = g.profile_end()
    g.close()
    assert prof["gemm_stream"]["launches"] == len(streams)
    assert prof["gemm_stream"]["bytes"] == sum((rows + n) * k * 2 + 4 * rows * n for n, k in streams)
    assert prof["gemm_reg"]["launches"] == 1 and prof["gemm_reg"]["flops"] == 2.0 * rows * d * m.d_ffn
