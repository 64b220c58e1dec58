"""CPU: the sort's placement kernel has no static LDS. Its launch sizes the dynamic block to a
CU's whole LDS at some key counts, so a byte beside it would make those launches fail."""
import re
import subprocess

from test_kernel_resources import LLVM, kernel_metadata


def test_placement_has_no_lds_beside_its_slot_rows(tmp_path):
    kernel_metadata(tmp_path)                            # leaves the code object in dev.co
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(tmp_path / "dev.co")], check=True,
                           capture_output=True, text=True).stdout
    size, sizes = None, {}
    for line in notes.splitlines():
        m = re.match(r"\s*(?:- )?\.(group_segment_fixed_size|name):\s+(\S+)", line)
        if m and m.group(1) == "group_segment_fixed_size":
            size = int(m.group(2))                       # stands before the kernel's name
        elif m and "k_sort_place" in m.group(2):
            sizes[m.group(2)] = size
    assert sizes and set(sizes.values()) == {0}, sizes
