"""Names of the kernels a call enqueues, without running them: the call is
captured into a HIP graph, whose kernel nodes are read and which is never
launched."""
import ctypes


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", _Dim3), ("params", ctypes.c_void_p), ("shared", ctypes.c_uint)]


def _hip():
    # the runtime torch and the library share
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    hip = ctypes.CDLL(path)
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    return hip


def kernel_names(torch, call):
    """Mangled names of the kernels that call(stream) puts on stream, in order."""
    hip = _hip()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    s, graph = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p()

    def ok(status):
        assert status == 0, status

    ok(hip.hipStreamBeginCapture(s, 2))  # relaxed
    try:
        call(stream)
    finally:
        ok(hip.hipStreamEndCapture(s, ctypes.byref(graph)))
    try:
        n = ctypes.c_size_t()
        ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)))
        nodes = (ctypes.c_void_p * n.value)()
        ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)))
        names = []
        for node in nodes:
            p = _KernelNodeParams()
            ok(hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)))
            names.append(hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), s).decode())
        return names
    finally:
        ok(hip.hipGraphDestroy(graph))
