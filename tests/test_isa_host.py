"""The machine code of the built library keeps the wait states that gfx950 does not keep by itself (no GPU needed).

The result of a matrix product may be read by another unit only some wait states after the product: the number of its
passes (four cycles each) and four more for the 16-bit products, two for the fp32 ones.  The compiler puts them in where it
sees the reader, not where the reader stands inside inline assembly."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_21571_amd import _build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
WAIT = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_16x16x32_f16": 8, "v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_32x32x16_f16": 12,
        "v_mfma_f32_16x16x4_f32": 10}
REG = re.compile(r"\b([av])(?:(\d+)\b|\[(\d+):(\d+)\])")
LINE = re.compile(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):(.*)$")


def _regs(text):
    out = set()
    for bank, one, lo, hi in REG.findall(text):
        out.update((bank, i) for i in (range(int(lo), int(hi) + 1) if lo else [int(one)]))
    return out


def _kernels(listing):
    """(name, [(address, opcode, operands, rest of the line)]) of a disassembly."""
    name, body = None, []
    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.+)>:$", line)
        if head:
            if body:
                yield name, body
            name, body = head.group(1), []
            continue
        m = LINE.match(line)
        if m:
            body.append((int(m.group(3), 16), m.group(1), m.group(2), m.group(4)))
    if body:
        yield name, body


def _written_and_read(op, operands):
    first, _, rest = operands.partition(", ")
    if "store" in op or op.startswith("ds_write") or "lds_dword" in op:
        return set(), _regs(operands)
    if "swap" in op:
        return _regs(operands), _regs(operands)
    return _regs(first), _regs(rest)


def early_reads(listing):
    """[(kernel, address, wait states, reader)]: every path behind a product is followed until its result is ready."""
    found, products = [], 0
    for name, body in _kernels(listing):
        at = {a: i for i, (a, *_) in enumerate(body)}

        def target(rest):
            m = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>", rest)
            return at[body[0][0] + int(m.group(1) or "0", 16)]

        for i, (_, op, operands, _) in enumerate(body):
            if not op.startswith("v_mfma"):
                continue
            products += 1
            paths = [(i + 1, 0, _regs(operands.partition(", ")[0]))]
            while paths:
                j, waited, fresh = paths.pop()
                while fresh and waited < WAIT[op] and j < len(body):
                    a, o, ops, rest = body[j]
                    if o == "s_endpgm":
                        break
                    written, read = _written_and_read(o, ops)
                    if o.startswith("v_mfma"):  # (products in a chain have a rule of their own)
                        read = set()
                    if read & fresh:
                        found.append((name, hex(a), waited, o))
                    fresh = fresh - read - written
                    waited += int(ops) + 1 if o == "s_nop" else 1
                    if o == "s_branch":
                        j = target(rest)
                        continue
                    if o.startswith("s_cbranch"):
                        paths.append((target(rest), waited, fresh))
                    j += 1
    return found, products


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not os.path.exists(_build.LIB_PATH):
        _build.build()
    d = tmp_path_factory.mktemp("isa")
    lib = shutil.copy(_build.LIB_PATH, d)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)  # (leaves the code objects beside it)
    objects = sorted(f for f in os.listdir(d) if f.endswith("gfx950"))
    assert objects
    return [subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(d, f)], check=True, capture_output=True, text=True).stdout
            for f in objects]


def test_no_product_is_read_before_it_is_ready(listings):
    total = 0
    for text in listings:
        found, products = early_reads(text)
        assert not found, found[:8]
        total += products
    assert total > 1000


def test_the_check_sees_a_read_that_comes_too_early():
    def listing(nops, skip):
        ins = ["v_mfma_f32_32x32x16_f16 v[4:19], v[20:23], v[24:27], v[4:19]"]
        ins += ["s_cbranch_scc1 %d" % 0] if skip else []
        ins += ["s_nop %d" % nops, "v_max3_f32 v1, v7, v8, v9", "s_endpgm"]
        out, a = ["0000000000001000 <k>:"], 0x1000
        for n, s in enumerate(ins):
            to = " <k+0x%x>" % (4 * (len(ins) - 2)) if "cbranch" in s else ""
            out.append("\t%s // %012X: 00000000%s" % (s, a + 4 * n, to))
        return "\n".join(out)

    assert early_reads(listing(11, False)) == ([], 1)
    assert [f[2] for f in early_reads(listing(7, False))[0]] == [8]
    assert [f[2] for f in early_reads(listing(15, True))[0]] == [1]  # past the s_nop
