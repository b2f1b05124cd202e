"""Order of the training kernel's exchange between workgroups, read from the
instructions of the built library (no GPU needed).

One thread publishes the sums that every wave of its workgroup has stored, and
the reading of those that every wave has loaded. A wave's count of outstanding
memory operations is its own, so each wave has to wait for its own stores and
loads before the barrier that the publishing thread passes: a bare barrier
lets the count go out while another wave's stores are still on their way."""
import os
import re
import shutil
import subprocess

import pytest

from test_kernel_resources import LIB, LLVM, MAGIC, TARGET, TOOLS

OBJDUMP = os.path.join(LLVM, "llvm-objdump")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not all(os.path.exists(t) for t in TOOLS + [OBJDUMP]),
                                reason="needs the built library and the ROCm LLVM tools")


@pytest.fixture(scope="module")
def train_kernels(tmp_path_factory):
    """Instructions of the shared training kernels, by name."""
    d = tmp_path_factory.mktemp("codeobj")
    fat = d / "fatbin"
    subprocess.run([TOOLS[0], f"--dump-section=.hip_fatbin={fat}", LIB, str(d / "lib.so")], check=True,
                   capture_output=True)
    data = fat.read_bytes()
    starts = [m.start() for m in re.finditer(re.escape(MAGIC), data)] + [len(data)]
    out = {}
    for k in range(len(starts) - 1):
        b, co = d / f"bundle{k}", d / f"co{k}"
        b.write_bytes(data[starts[k]:starts[k + 1]])
        subprocess.run([TOOLS[1], "--unbundle", "--type=o", f"--targets={TARGET}", f"--input={b}", f"--output={co}"],
                       check=True, capture_output=True)
        if b"k_train" not in co.read_bytes():
            continue
        text = subprocess.run([OBJDUMP, "-d", str(co)], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name, _, body = block.partition(">:")
            if re.search(r"k_trainILi\d+ELb0E", name):
                out[name] = [line.split("//")[0].strip() for line in body.splitlines() if line.strip()]
    shutil.rmtree(d, ignore_errors=True)
    return out


def test_every_wave_waits_before_its_workgroup_is_counted(train_kernels):
    assert len(train_kernels) == 2  # both network widths
    for name, code in train_kernels.items():
        published = [i for i, ins in enumerate(code) if ins.startswith("buffer_wbl2")]
        assert len(published) >= 2, name  # the sums are written; the sums are read
        for i in published:
            barrier = max(j for j in range(i) if code[j].startswith("s_barrier"))
            for ins in reversed(code[:barrier]):
                if re.match(r"s_waitcnt .*vmcnt\(0\)", ins):
                    break
                assert not re.match(r"(global|buffer|flat)_(load|store|atomic)", ins), (name, ins)
