"""Inline assembly of the kernels tells the compiler every fixed register that it writes: one that is not
in the clobber list may hold a value of the compiler's own across the statement."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_19720_amd", "csrc")


def statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        for body in re.findall(r"\basm\s*(?:volatile)?\s*\((.*?)\);", open(path).read(), flags=re.S):
            yield os.path.basename(path), body


def test_fixed_registers_are_declared():
    seen = 0
    for name, body in statements():
        template = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)*)', body).group(1)
        clobbers = body.rsplit(":", 1)[1]
        for reg in ("m0", "vcc"):
            if re.search(r"(?:^|\\t|[\s\"])[sv]_\w+ (?:%\d+, )?" + reg + r"\b", template):
                seen += 1
                assert f'"{reg}"' in clobbers, f"{name}: asm writes {reg}: {body}"
    assert seen >= 4, "the direct loads into LDS set m0"
