"""What the device sources must not contain."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_15618_amd", "csrc")


def test_loads_are_known_to_the_compiler():
    """A load in an inline assembly statement of its own hands out a register whose data is still on its way: nothing keeps the compiler
    from copying it before the wait.  All loads go through builtins, so that it places the waits itself."""
    files = glob.glob(os.path.join(CSRC, "*"))
    assert len(files) > 5
    for f in files:
        for n, line in enumerate(open(f), 1):
            assert not re.search(r'asm\b.*"\s*(global|buffer|flat|scratch|ds|s)_(load|read)', line), f"{os.path.basename(f)}:{n}"
