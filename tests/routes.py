"""Which kernel libwd chooses for a configuration: its host side compiled into a library of its own that answers that."""
import collections
import ctypes
import os
import subprocess
import tempfile

Route = collections.namedtuple("Route", "kernel teams threads strips wide apart reach lds")
HERE = os.path.dirname(os.path.abspath(__file__))
_probe = None


def _load():
    global _probe
    if _probe is None:
        import paper_2108_13976_amd as wd
        from paper_2108_13976_amd import build

        wd.load_library()
        package = build.HERE
        with tempfile.TemporaryDirectory() as scratch:
            library = os.path.join(scratch, "route_probe.so")
            subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.HIPCC_FLAGS +
                           ["-O1", "-Wno-unused-function", "-I", build.CSRC, "-o", library, os.path.join(HERE, "route_probe.hip"),
                            "-L" + package, "-l:libwd.so", "-Wl,-rpath," + package], check=True, stderr=subprocess.DEVNULL)
            _probe = ctypes.CDLL(library)
    return _probe


def route(kw, recording=False):
    """The kernel that serves `kw` (arguments of TagEnvs), in single calls or in wd_rollout, and its geometry."""
    from paper_2108_13976_amd import binding

    args = {k: v for k, v in kw.items() if k not in ("device",)}
    args.setdefault("episode_length", 5)
    cfg = binding.make_config(**args)
    out = ctypes.create_string_buffer(128)
    rc = _load().wd_test_route(ctypes.byref(cfg), int(recording), out, len(out))
    assert rc == 0, (rc, kw)
    words = out.value.decode().split()
    return Route(words[0], *map(int, words[1:]))
