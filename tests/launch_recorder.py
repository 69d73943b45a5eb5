"""Runs a piece of Python against libpf.so on a host without a GPU and returns
the launches and attributes the library asked for (tests/hip_recorder.c)."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
R = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
R.rec_text.restype = ctypes.c_char_p
L = ctypes.CDLL(sys.argv[2])
vp, u64, u32, i32, f32 = ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int32, ctypes.c_float
class pf_table(ctypes.Structure):
    _fields_ = [(n, vp) for n in ("cell", "key", "blend", "occ", "stats")] + [
        ("log2_slots", u32), ("max_probe", u32), ("frac_bits", i32), ("sum_format", u32)]
class pf_key_params(ctypes.Structure):
    _fields_ = [("cam", f32 * 3), ("s", f32), ("seed", u64), ("idx_base", u64)]
class pf_view(ctypes.Structure):
    _fields_ = [(n, vp) for n in ("px", "py", "pz", "nx", "ny", "nz", "valid", "r", "g", "b", "key", "vflags", "slot",
                                  "r_out", "g_out", "b_out", "count_out")] + [
        ("cur", pf_table), ("prev", pf_table), ("kp", pf_key_params), ("n", u32), ("alpha_old", f32),
        ("temporal", i32), ("reserved", u32)]
def table(log2_slots, at=0x700000000000, fmt=0):
    t = pf_table()
    assert L.pf_table_carve(vp(at), u32(log2_slots), 1, u32(16), i32(24), ctypes.byref(t)) == 0
    t.sum_format = fmt
    return t
def launches():
    out = R.rec_text().decode()
    R.rec_clear()
    return out
p = [vp(0x600000000000 + (k << 36)) for k in range(20)]  # never read
"""


def record(tmp_path, code):
    """Stdout of `code` after the prelude."""
    lib = os.path.join(str(tmp_path), "librecorder.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-I/opt/rocm/include", "-o", lib,
                    os.path.join(HERE, "hip_recorder.c")], check=True)
    res = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code), lib,
                          os.path.join(ROOT, "paper_1902_05942_amd", "libpf.so")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return res.stdout
