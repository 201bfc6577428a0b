"""The Python binding's host side, without a GPU."""
import ctypes as C

import paper_1410_2569_amd as L


def test_state_buffers_leave_the_shared_python_api_alone():
    """A state's bytes object is made through Python's C API, whose function objects in
    ctypes.pythonapi are shared by the whole process: another module's prototype must neither be
    changed nor be used."""
    make = C.pythonapi.PyBytes_FromStringAndSize
    before = make.argtypes, make.restype
    try:
        make.argtypes, make.restype = [C.c_void_p, C.c_ssize_t], C.py_object
        blob, at = L.lbm._new_bytes(64)
        assert make.argtypes == [C.c_void_p, C.c_ssize_t]
        C.memmove(at, bytes(range(64)), 64)
        assert blob == bytes(range(64))
        make.argtypes, make.restype = None, C.c_int
        blob, at = L.lbm._new_bytes(40)
        assert make.restype is C.c_int and isinstance(blob, bytes) and len(blob) == 40
    finally:
        make.argtypes, make.restype = before
