"""The GM/GQ matrix kernels set the f32 rounding mode to "toward zero" around
their generation loop.  Nothing that rounds in f32 by itself may stand between
the two mode writes: no reciprocal and no conversion from f32, of which the
compiler makes an integer division.  Read from the assembly of the kernels,
compiled here with the library's flags."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_1307_5869_amd import build as B

SOURCES = ["k_gm.hip", "k_batch.hip"]


def _assembly(name):
    cmd = [B.HIPCC] + [f for f in B.FLAGS if f != "-fPIC"] + B.SOURCE_FLAGS[name] + \
          ["--cuda-device-only", "-S", "-x", "hip", os.path.join(B.CSRC, name), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


def test_no_division_under_the_rounding_mode():
    with ThreadPoolExecutor(2) as ex:
        texts = list(ex.map(_assembly, SOURCES))
    found = 0
    for text in texts:
        for name, body in re.findall(r"^(_Z\w+):[^\n]*\n(.*?)^\.Lfunc_end\d+:", text, flags=re.M | re.S):
            modes = [m.start() for m in re.finditer(r"s_setreg_imm32_b32 hwreg\(HW_REG_MODE, 0, 2\)", body)]
            if not modes:
                continue
            found += 1
            assert len(modes) % 2 == 0, name
            for a, b in zip(modes[::2], modes[1::2]):
                bad = re.findall(r"\bv_(?:rcp\w*|rcp_iflag\w*|cvt_[iu]32_f32|div_\w+)\b", body[a:b])
                assert not bad, (name, bad)
    assert found >= 8 * 3 * 2
