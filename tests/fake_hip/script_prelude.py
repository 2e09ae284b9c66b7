import ctypes as C
import os

import numpy as np

from paper_2505_14468_amd import binding as B

F = C.CDLL(os.environ["FAKE_HIP"])
F.fake_name.restype = C.c_char_p
F.fake_arg1.restype = C.c_void_p
F.fake_event_waits.restype = C.c_long
ctx = B.lora_ctx_create(0)
F.fake_reset()

_keep = []


def mem(nbytes):
    """Address of `nbytes` of zeros, 256-byte aligned, kept until the process ends (nothing runs that would use it)."""
    a = np.zeros(nbytes + 256, np.uint8)
    _keep.append(a)
    return (a.ctypes.data + 255) // 256 * 256


def say(what, value):
    F.fake_set(what.encode(), int(value))


def launched():
    """[(kernel name, (grid x, y, z), (block x, y, z))] since the last reset."""
    out = []
    for i in range(F.fake_launches()):
        d = (C.c_uint * 6)()
        F.fake_dims(i, d)
        out.append((F.fake_name(i).decode(), tuple(d[:3]), tuple(d[3:])))
    return out


def tables():
    """[(address, ticket)] of the table that each launch of the plan kernel was given."""
    out = []
    for i in range(F.fake_launches()):
        if "plan_apply_kernel" in F.fake_name(i).decode():
            a = F.fake_arg1(i)
            out.append((C.c_uint64.from_address(a).value, C.c_uint32.from_address(a + 16).value))
    return out


def read_table(i):
    """What the plan kernel of launch `i` does first: its word receives its ticket."""
    a = F.fake_arg1(i)
    C.c_uint32.from_address(C.c_uint64.from_address(a + 8).value).value = C.c_uint32.from_address(a + 16).value


def make_plan(ids, ntok, ranks, r_max=None, raw=False):
    ids, ntok, ranks = (np.asarray(v, np.int32) for v in (ids, ntok, ranks))
    r_max = int(ranks.max()) if r_max is None else r_max
    T = int(ntok.sum())
    n = B.lora_plan_bytes(len(ids), T, len(ranks), r_max)
    return B.lora_plan(ctx, ids, ntok, ranks, r_max, T, mem(n), n, 0, raw=raw)


def make_desc(plan, K, N, dtype=B.LORA_DTYPE_BF16, ws_bytes=None, X=None, adapters=True):
    es = 2 if dtype == B.LORA_DTYPE_BF16 else 4
    T, ld = plan.T, (N + 7) // 8 * 8
    if ws_bytes is None:
        ws_bytes = B.lora_linear_workspace_bytes_preferred(T, K, N, plan.r_max, dtype)
    tbl = B.make_adapter_table(plan.n_adapters, mem(8 * plan.n_adapters), mem(8 * plan.n_adapters), mem(4 * plan.n_adapters)) if adapters else None
    return B.make_linear_desc(dtype, K, N, mem(T * K * es) if X is None else X, K, mem(N * K * es), K,
                              mem(T * ld * es), ld, tbl, mem(ws_bytes) if ws_bytes else None, ws_bytes)
