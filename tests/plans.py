"""The launch plans of the library (host code, no GPU): what a call of given sizes is routed to."""
import ctypes as C

TILES = ("dma_32x128", "dma_64x128", "dma_128x128", "dma_128x256", "dma_256x256", "dma_128x96", "dma_128x192", "dma_256x192",
         "dma_192x256", "reg_64x128", "simt")
EIGHT_WAVEFRONTS = ("dma_256x256", "dma_256x192", "dma_192x256")
STAGGER, XCD_GROUP, STREAM_W = 1, 2, 8


class GemmPlan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("kind", "split_k", "frac_units", "flags")]

    @property
    def tile(self):
        return TILES[self.kind]

    def grid(self, m, n):
        """(rows of tiles, workgroups)"""
        bm, bn = (int(x) for x in self.tile.split("_")[1].split("x"))
        rows = -(-m // bm)
        return rows, rows * -(-n // bn) * self.split_k


CONSUMER, ONE_SLICE, OWN_LAUNCH, PRODUCT = 0, 1, 2, 3          # who adds the K slices up


def gemm_plan(m, n, k, slices_go_to=CONSUMER, dtype=0):
    """The plan of the gate / up projection inside a step; PRODUCT: of one whose fp32 product is stored; OWN_LAUNCH: of dkv_gemm."""
    from paper_2505_15781_amd import binding
    f = binding.lib._Z13dkv_gemm_planiiiii
    f.restype, f.argtypes = GemmPlan, [C.c_int] * 5
    return f(dtype, m, n, k, slices_go_to)


class AttnPlan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("use_mfma", "q_tiles", "splits", "tiles_per_split", "shared", "wide", "q_blocks", "ksplit_nq",
                                       "ksplit_waves", "q_groups")]

    @property
    def kernel(self):
        """'generic', 'wide', 'shared8', 'shared4', or 'ksplit' with query tiles per item and wavefronts, e.g. 'ksplit2x8'"""
        if not self.use_mfma:
            return "generic"
        return "wide" if self.wide else f"shared{self.shared}" if self.shared else f"ksplit{self.ksplit_nq}x{self.ksplit_waves}"


def attn_plan(shape, max_rows_per_seq):
    from paper_2505_15781_amd import binding
    f = binding.lib._Z13dkv_attn_planiiiiiii
    f.restype, f.argtypes = AttnPlan, [C.c_int] * 7
    return f(shape.dtype, shape.batch, shape.n_q_heads, shape.n_kv_heads, shape.seq_len, shape.head_dim, max_rows_per_seq)


def attn_plan_within(partial_bytes, shape, max_rows_per_seq):
    """The plan whose records of key slices take at most `partial_bytes`."""
    from paper_2505_15781_amd import binding
    f = binding.lib._Z20dkv_attn_plan_withinmiiiiiii
    f.restype, f.argtypes = AttnPlan, [C.c_size_t] + [C.c_int] * 7
    return f(partial_bytes, shape.dtype, shape.batch, shape.n_q_heads, shape.n_kv_heads, shape.seq_len, shape.head_dim, max_rows_per_seq)


class HeadEpilogue(C.Structure):
    _fields_ = [("kind", C.c_int), ("out", C.c_void_p), ("head_part", C.c_void_p), ("head_tiles", C.c_int), ("mask_id", C.c_int),
                ("status", C.c_void_p)]


def launch_head(x, w, tile, mask_id, status, rows=None, logits=None):
    """The vocabulary projection with the softmax statistics in its epilogue, on a given tile kernel (K in one slice).
    Returns the records [m][column tiles][4] as int32 (max and sum are float bits, then the arg max)."""
    import torch
    from paper_2505_15781_amd import binding as b
    m, k = x.shape
    n = w.shape[0]
    bn = int(tile.split("x")[1])
    tiles = -(-n // bn)
    part = torch.full((m, tiles, 4), 0x7fc00123, dtype=torch.int32, device=x.device)
    ep = HeadEpilogue(2, b._ptr(logits), part.data_ptr(), tiles, mask_id, status.data_ptr())
    f = b.lib._Z20dkv_launch_gemm_headPKvS0_iPKiii8GemmPlanRK12GemmEpilogueP12ihipStream_t
    f.restype = C.c_int
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_int, GemmPlan, C.POINTER(HeadEpilogue), C.c_void_p]
    b._check(f(x.data_ptr(), w.data_ptr(), m, b._ptr(rows), n, k, GemmPlan(TILES.index(tile), 1, 0, 0), C.byref(ep), b._stream()))
    return part


STREAM_TILES = {"stream_256x96": 11, "stream_256x64": 12}      # kinds that only the planner hands out, for projections inside a step


def launch_stream(x, w, tile, split, rows=None, swiglu=False):
    """A projection of at most 256 rows on one of STREAM_TILES: fp32 [split][m][n], or bf16 [m][n / 2] with the SwiGLU epilogue;
    NaN where the launch writes nothing. `rows`: device count of rows, at most m."""
    import torch
    from paper_2505_15781_amd import binding as b
    (m, k), n = x.shape, w.shape[0]
    out = torch.full((m, n // 2) if swiglu else (split, m, n), float("nan"), dtype=torch.bfloat16 if swiglu else torch.float32, device=x.device)
    f = b.lib._Z15dkv_launch_gemmiPKvS0_PfiiPKiii8GemmPlanP12ihipStream_t
    f.restype = C.c_int
    f.argtypes = [C.c_int] + [C.c_void_p] * 3 + [C.c_int] * 2 + [C.c_void_p] + [C.c_int] * 2 + [GemmPlan, C.c_void_p]
    b._check(f(0, x.data_ptr(), w.data_ptr(), out.data_ptr(), m, m, b._ptr(rows), n, k,
               GemmPlan(STREAM_TILES[tile], split, 0, 4 if swiglu else 0), b._stream()))
    return out


def embed_norm(table, tokens, pos, seq, counts, gain, h, a, stamp, eps, step):
    """The row kernel that begins a step: rows of the embedding table into h, their RMSNorm into a."""
    import torch
    from paper_2505_15781_amd import binding as b
    f = b.lib._Z21dkv_launch_embed_normiP12ihipStream_tiiPKvPKiS4_S4_S4_PKfPfPvPiifi
    f.restype = C.c_int
    f.argtypes = [C.c_int, C.c_void_p, C.c_int, C.c_int] + [C.c_void_p] * 9 + [C.c_int, C.c_float, C.c_int]
    b._check(f(0 if table.dtype == torch.bfloat16 else 1, b._stream(), h.shape[0], h.shape[1], table.data_ptr(), tokens.data_ptr(), pos.data_ptr(),
               seq.data_ptr(), counts.data_ptr(), gain.data_ptr(), h.data_ptr(), a.data_ptr(), stamp.data_ptr(), tokens.shape[1], eps, step))


def gather_rows(src, picks, counts, dst):
    """dst[c] = src[picks[c]] for c below counts[1]."""
    import torch
    from paper_2505_15781_amd import binding as b
    f = b.lib._Z22dkv_launch_gather_rowsiP12ihipStream_tiPKvPKiS4_Pvi
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_void_p, C.c_int] + [C.c_void_p] * 4 + [C.c_int]
    b._check(f(0 if src.dtype == torch.bfloat16 else 1, b._stream(), dst.shape[0], src.data_ptr(), picks.data_ptr(), counts.data_ptr(),
               dst.data_ptr(), dst.shape[1]))
