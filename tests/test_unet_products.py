"""The matrix products of the U-Net kernels in the device assembly (no GPU;
compiles one source): where a 16x16x16 and a 16x16x32 product follow each other
on one accumulator, the compiler inserts no wait states and the hardware needs
five, so another product has to lie between them, also across a loop's edge."""
import os
import re
import subprocess

from paper_2603_19371_amd import build


def kernels(text):
    """name -> basic blocks, each (label, [(opcode, accumulator, source)], branch targets)."""
    out, name = {}, None
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = [("", [], [])]
        if name is None:
            continue
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            out[name].append((m.group(1), [], []))
        m = re.match(r"\s+v_mfma_(\w+) (\S+), \S+, \S+, (\S+)", line)
        if m:
            out[name][-1][1].append(m.groups())
        m = re.match(r"\s+s_c?branch\w* (\.LBB\w+)", line)
        if m:
            out[name][-1][2].append(m.group(1))
        if "s_endpgm" in line:
            out[name].append(("end", [], []))
    return out


def sequences(blocks):
    """The products of each block in order, and of the blocks that may follow
    one another directly (fallen through or branched to, products in neither)."""
    with_products = [b for b in blocks if b[1]]
    for b in with_products:
        yield b[1]
    for a in with_products:
        for b in with_products:
            yield a[1][-1:] + b[1][:1]


def test_another_product_lies_between_dependent_ones_of_two_kinds(tmp_path):
    out = tmp_path / "k_unet.s"
    subprocess.run([build._hipcc(), *build._flags(), "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "k_unet.hip"), "-o", out], check=True,
                   capture_output=True)
    seen = 0
    for name, blocks in kernels(out.read_text()).items():
        for seq in sequences(blocks):
            for (op, acc, _), (op2, _, src) in zip(seq, seq[1:]):
                seen += op != op2
                assert op == op2 or acc != src, (name, op, op2, acc)
    assert seen  # the convolution does alternate them
