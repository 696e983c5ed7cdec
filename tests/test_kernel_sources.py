"""CPU-only checks of rules that the kernels' sources keep because a compiler does not."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_07752_amd", "csrc")


def _arguments(text, start):
    """The arguments of the call whose opening parenthesis is at `start`."""
    depth, args, begin = 0, [], start + 1
    for i in range(start, len(text)):
        if text[i] in "([{":
            depth += 1
        elif text[i] in ")]}":
            depth -= 1
            if depth == 0:
                return [a.strip() for a in args + [text[begin:i]]]
        elif text[i] == "," and depth == 1:
            args.append(text[begin:i])
            begin = i + 1


def test_wide_stores_carry_no_scalar_offset():
    """A store of 12 or 16 bytes with a scalar offset may store a value that the next instruction writes into its first data register."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__builtin_amdgcn_raw_(?:ptr_)?buffer_store_(?:b96|b128)\s*\(", text):
            args = _arguments(text, m.end() - 1)
            assert len(args) == 5 and args[3] == "0", f"{os.path.basename(path)}: {args}"
            seen += 1
    assert seen >= 20
