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
