"""A HIP stream of a test's own, made and destroyed through the library's HIP
runtime (torch hands out streams of a pool, one after the other, and with them
the hardware queues they share: a test that took some would move the streams,
and so the queues, of those after it)."""
import contextlib
import ctypes


@contextlib.contextmanager
def hip_stream(flb):
    import torch
    hip = flb.lib()  # its symbols and those of what it links
    s = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(s), ctypes.c_uint(1)) == 0
    # (after a failure the stream is left, as its handle still names it)
    yield torch.cuda.ExternalStream(s.value)
    assert hip.hipStreamSynchronize(s) == 0
    assert hip.hipStreamDestroy(s) == 0
