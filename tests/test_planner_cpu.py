"""The rules by which projection and attention calls choose their kernels (host code)."""
import pytest

import dkv_inputs as D
from dkv_inputs.configs import BF16

from plans import CONSUMER, EIGHT_WAVEFRONTS, ONE_SLICE, OWN_LAUNCH, PRODUCT, STREAM_TILES, STREAM_W, attn_plan, attn_plan_within, gemm_plan


@pytest.mark.parametrize("m,n,k", [(2049, 512, 4096), (4096, 512, 4096), (2304, 3584, 18944), (3072, 1024, 8192), (5000, 1024, 4096)])
def test_k_is_sliced_at_thousands_of_rows_where_few_columns_leave_the_chip_idle(m, n, k):
    """In one slice the launch has fewer workgroups than the chip has compute units, or a last round that is nearly empty:
    1.15 to 1.6 times the time of the sliced launch."""
    p = gemm_plan(m, n, k)
    assert p.split_k > 1, (p.tile, p.split_k)


@pytest.mark.parametrize("m,n,k", [(6144, 24576, 4096), (12288, 37888, 3584), (4096, 12288, 4096)])
def test_k_is_not_sliced_where_the_tiles_fill_the_chip(m, n, k):
    assert gemm_plan(m, n, k).split_k == 1


@pytest.mark.parametrize("m,n,k,tile", [(294, 37888, 3584, "dma_192x256"), (384, 37888, 3584, "dma_192x256"), (640, 24576, 4096, "dma_192x256"),
                                        (640, 12288, 4096, "dma_128x256"), (512, 4096, 12288, "dma_256x256")])
def test_128x256_tiles_are_planned_for_one_round(m, n, k, tile):
    """A second round of them (444 and 480 workgroups) costs more than its K tiles; one round (240) is theirs."""
    assert gemm_plan(m, n, k).tile == tile


@pytest.mark.parametrize("m,n,k,tile", [(384, 37888, 3584, "dma_128x256"), (640, 24576, 4096, "dma_128x256"), (600, 22016, 4096, "dma_128x256"),
                                        (640, 24576, 5120, "dma_128x256"), (800, 18432, 6144, "dma_128x256"), (400, 37888, 3584, "dma_192x256"),
                                        (288, 37888, 8192, "dma_192x256"), (608, 22016, 11008, "dma_192x256")])
def test_a_further_round_of_128x256_tiles_is_cheap_where_the_product_is_stored(m, n, k, tile):
    """The charge of the test above is for epilogues that compute: dkv_gemm and the projections whose fp32 product a row kernel
    reads keep these tiles in their second round, up to the line where a third begins and to K = 6144."""
    assert gemm_plan(m, n, k, OWN_LAUNCH).tile == tile and gemm_plan(m, n, k, PRODUCT).tile == tile


@pytest.mark.parametrize("m,n,k", [(191, 32000, 3584), (191, 28672, 3584), (137, 28672, 2048)])
def test_of_two_plans_that_only_stream_the_one_with_less_work_is_taken(m, n, k):
    """Two slices of 192x256 and of 256x256 tiles, both as fast as the operands come: no padding to 256 rows."""
    p = gemm_plan(m, n, k)
    assert p.tile == "dma_192x256" and p.split_k == 2


@pytest.mark.parametrize("m,n,k,tile", [(33, 65536, 2048, "dma_64x128"), (64, 65536, 512, "dma_64x128"), (82, 126464, 512, "dma_192x256"),
                                        (100, 126464, 4096, "dma_128x256"), (163, 65536, 1024, "dma_192x256"), (378, 65536, 512, "dma_192x256")])
def test_vocabularies_that_only_stream(m, n, k, tile):
    """A 128x256 tile for 33 to 64 candidates has as little work on paper as two 64x128, but three quarters of it is padding."""
    assert gemm_plan(m, n, k, ONE_SLICE).tile == tile


@pytest.mark.parametrize("m,n,k", [(400, 4608, 3584), (700, 4608, 3584), (1024, 4608, 3584), (400, 12288, 4096)])
def test_a_projection_on_its_own_pays_for_the_reduction_of_its_slices(m, n, k):
    """dkv_gemm adds the slices up in a launch of its own, a step's row kernel while it reads the product: where the slices
    gain little (measured: 13 to 25 % lost with the reduction) only the step is sliced."""
    from paper_2505_15781_amd import binding as b
    assert gemm_plan(m, n, k, OWN_LAUNCH).split_k == 1 and b.lib.dkv_gemm_workspace_bytes(m, n, k, b.BF16) == 0
    assert gemm_plan(m, n, k, CONSUMER).split_k > 1
    assert gemm_plan(64, 4096, 12288, OWN_LAUNCH).split_k > 1              # a long K on few tiles: sliced either way


def test_the_streaming_hint_is_planned_only_for_tiles_that_follow_it():
    """The 8-wavefront tiles have no non-temporal loads: a plan with the flag would claim what the launch does not do."""
    asked = 0
    for n, k in [(12288, 4096), (24576, 4096), (37888, 3584), (126464, 4096), (152064, 3584), (3584, 18944)]:
        for m in range(1, 257):
            for slices in (CONSUMER, ONE_SLICE, OWN_LAUNCH):
                p = gemm_plan(m, n, k, slices)
                if p.flags & STREAM_W:
                    asked += 1
                    assert p.tile not in EIGHT_WAVEFRONTS, (m, n, k, p.tile)
                    assert p.grid(m, n)[0] == 1
    assert asked > 500


def test_one_row_of_wide_tiles_is_planned_up_to_256_rows_inside_a_step():
    """Both sides of each line: the row counts, who asks, and shapes whose tiles do not make whole rounds or whose K is short."""
    stream = set(STREAM_TILES.values())
    for n, k in [(24576, 4096), (3584, 18944), (4096, 12288)]:
        assert gemm_plan(128, n, k).kind not in stream and gemm_plan(257, n, k).kind not in stream
        assert gemm_plan(160, n, k).kind in stream and gemm_plan(256, n, k).kind in stream
        assert gemm_plan(256, n, k, PRODUCT).kind in stream and gemm_plan(257, n, k, PRODUCT).kind not in stream
        assert gemm_plan(256, n, k, OWN_LAUNCH).kind not in stream and gemm_plan(256, n, k, ONE_SLICE).kind not in stream
    for n, k in [(37888, 3584), (4096, 4096), (3584, 3584), (1024, 8192)]:
        assert all(gemm_plan(m, n, k).kind not in stream for m in range(129, 257)), (n, k)


def test_every_attention_kernel_is_planned_where_its_measurements_say():
    """Both sides of each line of the dispatch (bf16, head_dim 128)."""
    def kernel(batch, q_heads, kv_heads, seq_len, rows):
        return attn_plan(D.AttnUpdateShape(batch, q_heads, kv_heads, seq_len, 128, dtype=BF16), rows).kernel

    assert kernel(8, 32, 32, 1024, 64) == "ksplit2x4" and kernel(8, 32, 32, 1024, 65) == "shared8"          # four query tiles
    assert kernel(6, 32, 32, 768, 128) == "shared8" and kernel(5, 32, 32, 768, 128).startswith("ksplit")      # 192 blocks
    assert kernel(8, 32, 32, 767, 128) == "wide" and kernel(8, 32, 32, 768, 129) == "wide"                    # long, one block
    assert kernel(15, 32, 32, 768, 128) == "shared8" and kernel(16, 32, 32, 768, 128) == "shared4"            # 512 pairs
    assert kernel(16, 28, 4, 768, 129) == "wide" and kernel(8, 32, 32, 1024, 512) == "wide"


@pytest.mark.parametrize("batch,q_heads,kv_heads,seq_len,rows,kernel,splits", [
    (1, 32, 32, 512, 30, "ksplit1x8", 1), (4, 32, 32, 512, 32, "ksplit1x8", 1), (4, 32, 32, 512, 33, "ksplit2x8", 1),     # 32 items per XCD
    (1, 28, 4, 512, 73, "ksplit1x8", 1), (1, 28, 4, 512, 74, "ksplit2x8", 1), (1, 28, 4, 768, 140, "ksplit2x8", 1),       # 4 pairs
    (3, 28, 4, 512, 36, "ksplit1x8", 1), (3, 28, 4, 512, 37, "ksplit2x8", 1),                                             # 12
    (5, 28, 4, 512, 22, "ksplit1x8", 1), (5, 28, 4, 512, 23, "ksplit2x8", 1),                                             # 20
    (1, 28, 4, 512, 146, "ksplit2x8", 1), (1, 28, 4, 512, 147, "ksplit2x4", 1),                                           # 33 of two tiles
    (2, 32, 32, 736, 5, "ksplit1x8", 1), (2, 32, 32, 737, 5, "ksplit1x8", 3), (1, 32, 32, 737, 5, "ksplit1x8", 3),        # 24 key tiles
    (2, 32, 32, 1120, 20, "ksplit1x8", 2), (2, 32, 32, 1121, 16, "ksplit1x8", 3), (1, 32, 32, 1121, 20, "ksplit1x8", 3),
    (3, 28, 4, 1536, 16, "ksplit1x8", 2), (3, 28, 4, 1536, 19, "ksplit2x8", 3),                                           # slices on 12 pairs
    (5, 32, 32, 1024, 20, "ksplit2x8", 1), (4, 32, 32, 1121, 9, "ksplit1x8", 2), (1, 16, 16, 8192, 9, "ksplit1x8", 9),    # 16 items; long
    (3, 12, 12, 8192, 64, "ksplit2x8", 3), (2, 28, 4, 8192, 48, "ksplit2x8", 2), (8, 28, 4, 16384, 16, "ksplit2x8", 2),   # two tiles, slices
    (1, 4, 1, 4008, 131, "ksplit2x8", 3), (1, 4, 1, 3000, 131, "ksplit2x8", 1), (1, 7, 1, 7026, 153, "ksplit2x8", 3),     # rounds of slices
    (20, 16, 16, 150, 40, "ksplit2x4", 1), (21, 8, 8, 200, 40, "ksplit1x4", 1), (22, 8, 8, 200, 40, "ksplit2x4", 1),        # 64 of 4 wavefronts
    (1, 28, 4, 1024, 9, "ksplit1x8", 3), (1, 28, 4, 1025, 9, "ksplit1x8", 3), (1, 28, 4, 1536, 64, "ksplit1x8", 1)])      # fewer than 8 pairs
def test_key_split_items_hold_one_query_tile_while_each_has_a_compute_unit(batch, q_heads, kv_heads, seq_len, rows, kernel, splits):
    """Both sides of each line, which are counted on the fullest XCD."""
    p = attn_plan(D.AttnUpdateShape(batch, q_heads, kv_heads, seq_len, 128, dtype=BF16), rows)
    assert (p.kernel, p.splits) == (kernel, splits)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_key_slices_only_go_into_idle_compute_units(head_dim):
    """Over the range of the calls: up to 2000 keys sliced plans make no more workgroups than an XCD has units, never more than four
    rounds; no slice is empty, the wavefronts fit the number of items, and 1024 keys are no line for few pairs."""
    sliced = 0
    for batch in (1, 2, 3, 5, 8, 13, 16):
        for q_heads, kv_heads in ((32, 32), (28, 4), (24, 8), (8, 1), (12, 12)):
            per_xcd = -(-batch * kv_heads // 8)
            for seq_len in (33, 512, 767, 769, 1024, 1025, 1536, 2049, 4096, 16384, 60000):
                for rows in (1, 2, 5, 9, 16, 17, 33, 64, 65, 100, 146, 147, 400):
                    p = attn_plan(D.AttnUpdateShape(batch, q_heads, kv_heads, seq_len, head_dim, dtype=BF16), min(rows, seq_len))
                    if not p.ksplit_nq:
                        continue
                    assert p.q_groups == -(-p.q_tiles // p.ksplit_nq) and (p.ksplit_waves == 8) == (per_xcd * p.q_groups <= 32 or p.splits > 1)
                    tiles = -(-seq_len // 32)
                    assert (p.splits - 1) * p.tiles_per_split < tiles <= p.splits * p.tiles_per_split
                    if p.splits > 1:
                        sliced += 1
                        assert per_xcd * p.q_groups * p.splits <= (32 if seq_len <= 2048 else 128) and tiles * head_dim >= 24 * 128
    assert sliced > 500
    small, large = (attn_plan(D.AttnUpdateShape(1, 28, 4, n, 128, dtype=BF16), 64) for n in (1024, 1025))
    assert (small.kernel, small.splits) == (large.kernel, large.splits)


def test_every_call_has_a_plan_within_the_static_scratch():
    """dkv_attn_update_static refuses no call for its size: where the records of the plan exceed its array, the plan within it."""
    from paper_2505_15781_amd import binding as b
    limit, shrunk = b.STATIC_SCRATCH_BYTES, 0
    for batch in (1, 2, 4, 7, 16, 31):
        for q_heads, kv_heads in ((32, 32), (28, 4), (56, 8), (8, 1), (3, 1), (190, 38)):
            for seq_len in (768, 1543, 2211, 5749, 15590, 40156):
                for rows in (1, 4, 7, 16, 26, 49, 115, 300):
                    s = D.AttnUpdateShape(batch, q_heads, kv_heads, seq_len, 128, dtype=BF16)
                    p, free = attn_plan_within(limit, s, rows), attn_plan(s, rows)
                    record = batch * -(-p.q_tiles * 16 // (q_heads // kv_heads)) * q_heads * (128 + 4) * 4
                    assert p.splits == 1 or record * p.splits <= limit
                    fits = free.splits == 1 or record * free.splits <= limit
                    assert not fits or (p.kernel, p.splits) == (free.kernel, free.splits)
                    shrunk += not fits
    assert shrunk > 50
