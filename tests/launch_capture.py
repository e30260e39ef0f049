"""The launches a call enqueues, read from a stream capture (nothing runs)."""
import ctypes


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class KernelNode(ctypes.Structure):          # hipKernelNodeParams
    _fields_ = [("block", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", Dim3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def launches(lib, call):
    """(call(stream)'s result, [(grid.x, threads per block)]) in the order enqueued, all on one stream."""
    vp = ctypes.c_void_p

    def hip(name, *args):
        fn = getattr(lib, name)
        fn.restype = ctypes.c_int
        rc = fn(*args)
        assert rc == 0, (name, rc)

    s, graph, n = vp(), vp(), ctypes.c_size_t()
    hip("hipStreamCreate", ctypes.byref(s))
    try:
        hip("hipStreamBeginCapture", s, ctypes.c_int(1))           # thread-local
        try:
            rc = call(s)
        finally:
            hip("hipStreamEndCapture", s, ctypes.byref(graph))
        out = []
        hip("hipGraphGetNodes", graph, vp(), ctypes.byref(n))
        nodes = (vp * max(1, n.value))()
        hip("hipGraphGetNodes", graph, nodes, ctypes.byref(n))
        for m in range(n.value):
            p = KernelNode()
            hip("hipGraphKernelNodeGetParams", vp(nodes[m]), ctypes.byref(p))
            out.append((p.grid.x, p.block.x * p.block.y * p.block.z))
        hip("hipGraphDestroy", graph)
    finally:
        hip("hipStreamDestroy", s)
    return rc, out
