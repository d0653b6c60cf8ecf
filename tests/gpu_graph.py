"""The kernels a library call launches, by name: the call is captured into a
HIP graph, which is printed and not run (for tests of which kernel a size
takes)."""
import ctypes
import os
import re
import tempfile

import torch

from paper_2211_15716_amd import igg

THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal
VERBOSE = 1       # hipGraphDebugDotFlagsVerbose


def kernels(call):
    """Names (mangled) of the kernels `call` launches on the current stream."""
    return [name for name, _ in launches(call)]


def launches(call):
    """(mangled name, work-groups in x) of the kernels `call` launches."""
    hip = igg.load()  # resolves the runtime's symbols too
    stream = torch.cuda.Stream()
    handle, graph = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(handle, THREAD_LOCAL) == 0
        try:
            call()
        finally:
            rc = hip.hipStreamEndCapture(handle, ctypes.byref(graph))
    assert rc == 0
    fd, path = tempfile.mkstemp(suffix=".dot")
    os.close(fd)
    try:
        assert hip.hipGraphDebugDotPrint(graph, path.encode(), VERBOSE) == 0
        with open(path) as f:
            text = f.read()
    finally:
        assert hip.hipGraphDestroy(graph) == 0
        os.unlink(path)
    found = re.findall(r"\{ID \| \d+ \| (\S+?)\\<\\<\\<\((\d+),", text)
    return [(name, int(groups)) for name, groups in found]
