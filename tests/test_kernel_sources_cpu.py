"""Rules that the kernel sources set themselves and no run can show."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_09190_amd", "csrc")


def _code(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def test_inline_assembly_maximum_never_feeds_a_lane_exchange():
    """max_abs is inline assembly: its result passes through an ordinary
    instruction before another lane reads it, and none of its arguments comes
    from a matrix-core product directly."""
    src = _code("kernels_gram.hip")
    uses = [m.start() for m in re.finditer(r"\bmax_abs\(", src)]
    assert len(uses) == 4   # the definition, two running maxima, and their join
    exchange = r"(?:wave_max_f64|row_perm_f64<[^>]*>|lane_pair\w*<[^>]*>|__shfl\w*|pair)\(\s*max_abs\("
    assert not re.search(exchange, src)
    assert not re.search(r"max_abs\(\s*(?:mfma64|a\[)", src)
