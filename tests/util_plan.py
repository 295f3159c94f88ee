"""Which kernels of the many-row path a call takes (host only: the cost models look at shapes alone)."""
import ctypes as C

import paper_2510_15312_amd as vf

GEMMS = ["qkv", "o", "gateup", "down", "head", "topk"]
SHAPES = ["T16x16", "T16x8", "T8x8", "S4x2", "S4x4", "S4x5", "S8x4", "S8x5", "S16x5", "S24x5", "S8x3", "S16x5W4"]
EPILOGUES = ["partial", "split", "qkv", "swiglu", "topk"]


def gemm_plan(cfg, gemm, rows, top_k=1):
    """(kernel, K splits, epilogue) of a GEMM of a vf_config at a number of rows."""
    out = (C.c_int32 * 4)()
    vf.binding._check(vf.lib.vf_debug_gemm_plan(C.byref(cfg), GEMMS.index(gemm) + (top_k - 1 if gemm == "topk" else 0), rows, out))
    assert out[3], f"{gemm} of {rows} rows: the partial sums do not fit"
    return SHAPES[out[0]], out[1], EPILOGUES[out[2]]


def attention_plan(cfg, lens, rows):
    """(pages of a part, parts merged): 0 pages: the kernel for few items."""
    n, out = len(lens), (C.c_int32 * 2)()
    arr = C.c_int32 * n
    vf.binding._check(vf.lib.vf_debug_attention_plan(C.byref(cfg), n, arr(*[int(x) for x in lens]), arr(*[int(x) for x in rows]), out))
    return out[0], bool(out[1])


def attention_reads_ahead(cfg, lens, rows):
    """Whether the kernel for few items reads the output projection's weights ahead."""
    n, out = len(lens), (C.c_int32 * 1)()
    arr = C.c_int32 * n
    vf.binding._check(vf.lib.vf_debug_attention_reads_ahead(C.byref(cfg), n, arr(*[int(x) for x in lens]), arr(*[int(x) for x in rows]), out))
    return bool(out[0])


def persistent_plan(cfg, rows):
    """(which persistent kernel a vf_verify of so many rows takes, grid barriers of its launch)."""
    out = (C.c_int32 * 2)()
    vf.binding._check(vf.lib.vf_debug_persistent_plan(C.byref(cfg), rows, out))
    return [None, "pass", "layers"][out[0]], out[1]
