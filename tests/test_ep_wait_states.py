"""Wait states of the tally kernels' vector code (csrc/ep_kernels.hip compiled
to gfx950 assembly here).  A vector instruction that reads a scalar register
which a vector instruction wrote (a carry or a compare mask) needs two wait
states between them on this target; the compiler keeps them in its own code, and
inline assembly has to keep them itself."""

import re
import subprocess

import pytest

from paper_1511_07658_amd import build as B

TWO_RESULTS = ("v_mad_u64_u32", "v_mad_i64_i32", "v_add_co", "v_addc_co", "v_sub_co", "v_subb_co", "v_subrev_co",
               "v_div_scale")


def scalars(operand):
    """The 32-bit scalar registers that an operand names."""
    if operand in ("vcc", "vcc_lo", "vcc_hi"):
        return {"vcc_lo", "vcc_hi"} if operand == "vcc" else {operand}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return {f"s{i}" for i in range(int(m.group(1)), int(m.group(2)) + 1)}
    return {operand} if re.fullmatch(r"s\d+", operand) else set()


def short_waits(lines, need=2):
    """(line, wait states) of every read that comes too soon after its write."""
    age, bad, reads = {}, [], 0     # register -> wait states since a vector instruction wrote it
    for line in lines:
        code = line.split(";")[0].strip()
        if not code or code.startswith(".") or code.endswith(":"):
            continue
        name, _, rest = code.partition(" ")
        states = int(rest.strip(), 0) + 1 if name == "s_nop" else 1
        ops = [o.strip(" -|") for o in re.split(r",\s*(?![^\[]*\])", rest)]
        written = set()
        if name.startswith("v_"):
            ndst = 2 if name.startswith(TWO_RESULTS) else 1
            written = set().union(*(scalars(o) for o in ops[:ndst]))
            read = set().union(*(scalars(o.split()[0]) for o in ops[ndst:] if o))
            reads += len(read & age.keys())
            bad += [(line.strip(), age[r]) for r in read if age.get(r, need) < need]
        age = {r: a + states for r, a in age.items()}
        age.update({r: 0 for r in written})
        if name.startswith("s_"):
            age = {r: a for r, a in age.items() if r not in scalars(ops[0])}   # rewritten by a scalar instruction
    return bad, reads


def test_the_count_of_wait_states():
    write, read = "v_mad_u64_u32 v[0:1], s[4:5], v2, s6, v[0:1]", "v_cndmask_b32 v3, 0, 1, s[4:5]"
    assert short_waits([write, read])[0] and short_waits([write, "s_nop 0", read])[0]
    assert not short_waits([write, "s_nop 1", read])[0]
    assert not short_waits([write, "v_mov_b32_e32 v9, v8", "s_nop 0", read])[0]
    assert short_waits(["v_cmp_gt_u64_e32 vcc, v[0:1], v[2:3]", "v_cndmask_b32_e32 v1, v2, v3, vcc"])[0]


@pytest.mark.skipif(not B.os.path.exists(B.HIPCC), reason="needs hipcc")
def test_no_scalar_is_read_too_soon(tmp_path):
    out = tmp_path / "ep.s"
    subprocess.run([B.HIPCC, *B.HIP_FLAGS, "-S", "--cuda-device-only", B.os.path.join(B.CSRC, "ep_kernels.hip"),
                    "-o", str(out)], check=True, stderr=subprocess.DEVNULL, timeout=300)
    bad, reads = short_waits(out.read_text().splitlines())
    assert reads > 20       # the carries of the products are among them
    assert not bad, (len(bad), bad[:5])
