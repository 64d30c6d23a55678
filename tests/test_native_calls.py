"""The Python binding's native call module (_skelcall), on the CPU: what it hands on
and what it leaves to the general path.  Each check runs in a process of its own,
since the module's state is the process's."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(code):
    res = subprocess.run([sys.executable, "-c", textwrap.dedent(code)], cwd=ROOT,
                         capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout


def test_exception_of_the_stream_query_is_raised():
    """An interrupt that arrives while the current stream is queried is not lost."""
    run("""
        import ctypes as C
        import paper_1405_2915_amd as skel
        lib = skel.load_library()
        call = skel._call
        names = [n for n in ("skel_map", "skel_reduce", "skel_mapreduce", "skel_mapoverlap1d",
                 "skel_mapoverlap1d_backward", "skel_mapoverlap2d_fields",
                 "skel_mapoverlap2d_fields_backward", "skel_scan", "skel_scan_rows",
                 "skel_reduce_segments")]
        def interrupted():
            raise KeyboardInterrupt
        class Box:
            handle = 1
        call.bind(Box, interrupted, {n: C.cast(getattr(lib, n), C.c_void_p).value for n in names})
        try:
            call.reduce(0, Box(), Box(), -1, None)
        except KeyboardInterrupt:
            pass
        else:
            raise SystemExit("the interrupt was dropped")
        assert call.reduce("no integer", Box(), Box(), -1, None) is None
    """)


def test_module_is_named_for_the_interpreter():
    out = run("""
        import sysconfig
        import paper_1405_2915_amd as skel
        skel.load_library()
        print(skel._call.__file__.endswith("_skelcall" + sysconfig.get_config_var("EXT_SUFFIX")))
    """)
    assert out.strip() == "True"


def test_general_path_without_the_module():
    """A library built without the module is loaded, and calls reach it through ctypes."""
    run("""
        import sys
        sys.modules["paper_1405_2915_amd._skelcall"] = None  # "not installed"
        import paper_1405_2915_amd as skel
        skel.load_library()
        assert skel._call.scan(1, 2, 3) is None
        c = skel.Container.__new__(skel.Container)
        c.handle = 1
        try:
            skel.skel_reduce(skel.SUM, c, c)
        except skel.SkelError as e:
            assert e.status == skel.E_NOINIT, e
        else:
            raise SystemExit("no error")
        c.handle = None
    """)


def test_allocator_callbacks_are_kept():
    """Initialising again hands the library the same callbacks: containers made before
    still hold their addresses."""
    run("""
        import ctypes as C, gc
        import paper_1405_2915_amd as skel
        seen = []
        class Lib:
            def skel_init(self, device, allocator):
                a = C.cast(allocator, C.POINTER(skel._Allocator)).contents
                seen.append((C.cast(a.alloc, C.c_void_p).value, C.cast(a.free, C.c_void_p).value))
                return skel.OK
        skel.load_library = lambda: Lib()
        skel.torch.cuda.init = skel.torch.cuda.set_device = lambda *a: None
        for _ in range(5):
            skel._init_device(0, "torch")
            gc.collect()
        assert len(set(seen)) == 1, seen
    """)
