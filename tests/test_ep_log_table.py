"""The tally kernel's table of interval logarithms, recomputed with 60 digits."""
import re
from decimal import Decimal, localcontext
from pathlib import Path

CSRC = Path(__file__).resolve().parents[1] / "paper_1511_07658_amd" / "csrc"


def test_every_entry_is_the_rounded_value():
    entries = re.findall(r"\{(\S+), (\S+)\}", "".join(
        line for line in (CSRC / "ep_log_table.inc").read_text().splitlines(True) if not line.startswith("//")))
    assert len(entries) == 256
    with localcontext() as ctx:
        ctx.prec = 60
        for i, (inv, m2log) in enumerate(entries):
            # the first interval is referred to 1/2 and the last to 1
            c = Decimal(1) / 2 if i == 0 else Decimal(1) if i == 255 else Decimal(2 * i + 513) / 1024
            assert float.fromhex(inv) == float(1 / c), i
            # rounded once, from the rounded reciprocal itself
            want = 2 * Decimal(float.fromhex(inv)).ln()
            # the first is twice the kernel's ln 2, the same number
            assert float.fromhex(m2log) == float(want), i
