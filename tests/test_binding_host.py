"""The binding's marshalling module without a device: a call with a number of words that no entry point takes is refused with the
interpreter lock held."""
import os
import subprocess
import sys

from paper_2508_02932_amd import build

CODE = """
import ctypes, importlib.machinery, importlib.util, threading, torch
path = {path!r}
spec = importlib.util.spec_from_file_location("_plora_binding", path, loader=importlib.machinery.ExtensionFileLoader("_plora_binding", path))
mod = importlib.util.module_from_spec(spec)
spec.loader.exec_module(mod)
words = []
entry = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_uint64] * 5)(lambda *a: words.append(a) or 7)
address = ctypes.cast(entry, ctypes.c_void_p).value
assert mod.call(address, "ddddd", 1, 2, 3, 4, 5) == 7 and words == [(1, 2, 3, 4, 5)]
for n in (0, 1, 4, 6, 7, 15, 16):
    try:
        mod.call(address, "d" * n, *range(n))
    except RuntimeError as e:
        assert "arguments" in str(e)
    else:
        raise AssertionError(n)
    t = threading.Thread(target=lambda: words.append(n))
    t.start()
    t.join()
    assert words.pop() == n and len(words) == 1
print("ok")
"""


def test_unsupported_number_of_words():
    if not os.path.exists(build.BINDING):
        build.build_binding()
    run = subprocess.run([sys.executable, "-c", CODE.format(path=build.BINDING)], capture_output=True, text=True, timeout=600)
    assert run.returncode == 0 and run.stdout.strip() == "ok", (run.returncode, run.stdout, run.stderr[-2000:])
