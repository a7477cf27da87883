"""The setup's last kernel hands its ticket to the host only after every wave's stores."""
import os
import re
import subprocess

import pytest

from paper_1410_2240_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def kernel_instructions(asm, name):
    body = re.search(rf"^_ZN\w*{name}\w*:.*?s_endpgm", asm, flags=re.S | re.M).group(0)
    return [m.group(1) for m in re.finditer(r"^\t([a-z]\w+[^\n;]*)", body, flags=re.M)]


def test_waves_wait_for_their_stores_before_the_ticket(tmp_path):
    """In the code built for k_coarse_setup each wave waits for its stores (vmcnt 0) between
    the last of them and the barrier that the ticket's wave passes: the barrier alone does
    not order them, and the host reads the ticket as the end of the setup."""
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = tmp_path / "mg_tail.s"
    flags = [x for x in build.HIPCC_FLAGS if x != "-shared"]
    subprocess.run([hipcc, *flags, "-w", f"-I{build.INCLUDE}", f"-I{build.CSRC}", "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "mg_tail.hip"), "-o", str(out)], check=True)
    code = kernel_instructions(out.read_text(), "k_coarse_setup")
    ticket = max(i for i, x in enumerate(code) if x.startswith("global_store") and "sc0 sc1" in x)
    barrier = max(i for i, x in enumerate(code[:ticket]) if x.startswith("s_barrier"))
    stores = [i for i, x in enumerate(code[:barrier]) if x.startswith(("global_store", "flat_store"))]
    assert len(stores) >= 4   # the pseudo-inverse's among them
    waits = [i for i, x in enumerate(code[:barrier]) if x.startswith("s_waitcnt") and "vmcnt(0)" in x]
    assert waits and waits[-1] > stores[-1]
