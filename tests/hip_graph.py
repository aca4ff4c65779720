"""The kernels that a call enqueues, by name: the call is captured into a HIP graph, which is read
and thrown away (nothing runs)."""
import ctypes


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def kernels_of(torch, melt, call):
    """Names (mangled) of the kernels of one call, in launch order; "" for a node of another kind."""
    hip = ctypes.CDLL(melt.load_library()._name)       # its symbols include those of the HIP runtime it is linked to
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]

    def ok(status):
        assert status == 0, f"HIP status {status}"

    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    handle, graph = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p()
    ok(hip.hipStreamBeginCapture(handle, 1))           # this thread's calls only
    try:
        with torch.cuda.stream(stream):
            call()
    finally:
        status = hip.hipStreamEndCapture(handle, ctypes.byref(graph))
    ok(status)
    try:
        count = ctypes.c_size_t()
        ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(count)))
        nodes = (ctypes.c_void_p * count.value)()
        ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)))
        names = []
        for node in nodes:
            kind, p = ctypes.c_int(), _KernelNodeParams()
            ok(hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)))
            if kind.value != 0:
                names.append("")
                continue
            ok(hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)))
            names.append(hip.hipKernelNameRefByPtr(p.func, None).decode())
        return names
    finally:
        ok(hip.hipGraphDestroy(graph))
