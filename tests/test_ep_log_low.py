"""What the tally kernel's interval logarithms lack, recomputed with 60 digits."""
import re
from decimal import Decimal, localcontext
from pathlib import Path

CSRC = Path(__file__).resolve().parents[1] / "paper_1511_07658_amd" / "csrc"


def test_every_entry_is_the_rest_of_the_rounded_value():
    entries = re.findall(r"\{(\S+), (\S+)\}", (CSRC / "ep_log_table.inc").read_text().split("decimal digits).")[1])
    low = re.findall(r"(-?0x\S+),", (CSRC / "ep_log_low.inc").read_text())
    assert len(entries) == len(low) == 256
    with localcontext() as ctx:
        ctx.prec = 60
        for (inv, m2log), rest in zip(entries, low):
            want = 2 * Decimal(float.fromhex(inv)).ln() - Decimal(float.fromhex(m2log))
            assert float.fromhex(rest) == float(want), (inv, m2log)
    # the kernel's constant for 2 ln 2 is the first interval's
    assert f"kTwoLn2Low = {low[0]};" in (CSRC / "ep_kernels.hip").read_text()
