"""Order of memory accesses at the end of the group serving kernels, checked
in the code that the compiler makes of them (no GPU). Four waves write a
block's results and its last one raises the request's flag for all of them, so
each wave must have waited for its own stores -- the request's results and the
count of rays whose spill chunks ran out -- before it counts itself off in
LDS: the release of the last wave waits for that wave's stores only. And in
every serving kernel the L2 write-back of a release has to be waited for
before the chunk is counted off its request."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1310_1854_amd import build_lib

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def _code(tmp_path, kernel):
    out = str(tmp_path / "serve.s")
    flags = [f for f in build_lib.FLAGS if f != "-shared"]
    subprocess.run(["hipcc", "-S", "--cuda-device-only"] + flags + [os.path.join(build_lib.CSRC, "serve.hip"), "-o", out],
                   check=True, capture_output=True)
    kernels = re.findall(rf"^(\S*{kernel}\S*):(.*?)s_endpgm", open(out).read(), re.M | re.S)
    assert len(kernels) == 3, [k for k, _ in kernels]
    return [(name, [ln.split(";")[0].strip() for ln in code.splitlines()]) for name, code in kernels]


@pytest.mark.parametrize("kernel", ["k_serve_group", "k_serveI"])
def test_write_backs_are_waited_for(tmp_path, kernel):
    for name, code in _code(tmp_path, kernel):
        backs = [i for i, ln in enumerate(code) if ln == "buffer_wbl2 sc1"]
        assert backs, name
        for i in backs:
            after = [ln for ln in code[i + 1:] if re.match(r"(flat|global)_(store|atomic)|s_waitcnt.*vmcnt\(0\)", ln)]
            assert after[0].startswith("s_waitcnt"), f"{name}: the chunk is counted with a write-back in flight"


def test_every_wave_waits_for_its_stores_before_it_is_counted(tmp_path):
    for name, code in _code(tmp_path, "k_serve_group"):
        count = [i for i, ln in enumerate(code) if ln.startswith("ds_add_rtn_u32")]
        assert len(count) == 1, name   # the waves of the block, as they end
        before = code[:count[0]]
        store = [i for i, ln in enumerate(before) if re.match(r"(flat|global)_(store|atomic)", ln)]
        assert store, name
        waits = [i for i, ln in enumerate(before) if ln.startswith("s_waitcnt") and "vmcnt(0)" in ln]
        assert waits and waits[-1] > store[-1], f"{name}: a wave is counted with stores in flight"
