"""What the library launches, seen from the host (no GPU)."""
from launch_recorder import record

VIEWS = """
def view(n, log2_slots, at):
    d = pf_view(*[q.value + at for q in p[:17]])
    d.cur, d.prev = table(log2_slots, 0x700000000000 + 256 * at), table(log2_slots, 0x780000000000 + 256 * at)
    d.kp.s, d.n, d.alpha_old, d.temporal = 0.01, n, 0.2, 1
    return d
def filter_views(sizes, block, agg, grid_per_cu=0):
    views = (pf_view * len(sizes))(*[view(n, 20, k << 28) for k, n in enumerate(sizes)])
    ws = vp(0x500000000000)
    assert L.pf_filter_views(views, u32(len(sizes)), u32(block), u32(agg), u32(grid_per_cu), ws,
                             ctypes.c_size_t(1 << 30), None) == 0
    return launches()
"""


def test_views_lookup_is_a_launch_of_its_own(tmp_path):
    """The insert's registers leave the persistent launch half the wavefronts a
    compute unit holds; the lookup, bound by its gathers, is not part of it."""
    out = record(tmp_path, VIEWS + "print(filter_views([1000000, 30], 1024, 1024))").splitlines()
    kinds = [line.split()[0] for line in out if line]
    names = [line.split()[2] for line in out if line]
    assert kinds == ["launch", "cooperative", "launch"]
    assert "views_kernel" in names[1] and "lookup" in names[2]


def test_large_lds_is_allowed_on_every_device(tmp_path):
    """More than 64 KB of dynamic LDS is an attribute of a kernel on a device: a
    process that goes on to a second device sets it there too."""
    out = record(tmp_path, """
    t = table(22)
    class pf_mlp(ctypes.Structure):
        _fields_ = [(n, vp) for n in ("w", "m", "v", "wb", "partial", "loss")] + [("max_batch", u32), ("pad", u32)]
    class pf_geometry(ctypes.Structure):
        _fields_ = [(n, vp) for n in ("key", "px", "py", "pz", "nx", "ny", "nz")] + [("cam", f32 * 3), ("pad", u32)]
    net, geo = pf_mlp(), pf_geometry(*p[:7])
    assert L.pf_mlp_carve(vp(0x500000000000), u32(1024), ctypes.byref(net)) == 0
    for device in (0, 1):
        R.rec_set_device(device)
        for _ in range(2):
            assert L.pf_insert_accumulate(ctypes.byref(t), *p[:6], u64(1 << 21), u32(0), None) == 0
            assert L.pf_insert_accumulate_binned(ctypes.byref(t), *p[:6], u64(1 << 21), p[6],
                                                 ctypes.c_size_t(1 << 40), None) == 0
            assert L.pf_mlp_train_step(ctypes.byref(net), ctypes.byref(t), ctypes.byref(geo), p[7], p[8], p[9],
                                       u32(1024), u64(1), u32(1), f32(0.1), None) == 0
            assert L.pf_mlp_infer(ctypes.byref(net), ctypes.byref(geo), p[7], p[8], u64(1000), *p[9:12], None) == 0
    print(launches())
    """)
    rows = [line.split() for line in out.splitlines() if line]
    large = {(row[1], row[2]) for row in rows if row[0] == "launch" and int(row[5]) > 64 << 10}
    assert {device for device, _ in large} == {"0", "1"} and len(large) >= 8
    for row in rows:
        if row[0] == "attribute":
            large.discard((row[1], row[2]))
        elif row[0] == "launch":
            assert (row[1], row[2]) not in large, f"{row[2]} on device {row[1]} before its attribute"
    assert not large
    attributes = [row for row in rows if row[0] == "attribute"]
    assert len(attributes) == len({tuple(row) for row in attributes}), "set once"


def test_views_grid_is_the_devices_own(tmp_path):
    """The recorder's devices have 256 and 128 compute units, whose LDS holds two
    workgroups each."""
    out = record(tmp_path, VIEWS + """
for device in (0, 1, 0):
    R.rec_set_device(device)
    print(filter_views([100000], 512, 512))
""")
    grids = [int(line.split()[3]) for line in out.splitlines() if line.startswith("cooperative")]
    assert grids == [512, 256, 512]


def test_views_grid_of_threads_that_call_together(tmp_path):
    """A second thread must not launch with what the first has only half found out:
    a cooperative grid that is not resident at once would wait for itself."""
    out = record(tmp_path, VIEWS + """
import threading, time
launches = lambda: None
a = threading.Thread(target=filter_views, args=([100000], 64, 64))
a.start()
time.sleep(0.05)
b = threading.Thread(target=filter_views, args=([100000], 64, 64))
b.start()
a.join(), b.join()
print(R.rec_text().decode())
""")
    grids = [int(line.split()[3]) for line in out.splitlines() if line.startswith("cooperative")]
    assert grids == [512, 512]
