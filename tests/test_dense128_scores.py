"""The score products of the 128-dim dense kernel are inline assembly, so the compiler
does not know that a 32x32x16 product takes up to 18 wait states to write its
registers.  This walks the built kernels' own instructions from every such product,
along every branch, and finds none that touches those registers too early: whatever
order and registers the compiler chose, the distance is there."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_20125_amd", "libheadcast.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
OBJCOPY = "/opt/rocm/llvm/bin/llvm-objcopy"
WAIT = 18          # wait states until a product's result may be read or overwritten
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def device_objects(tmp):
    """The gfx950 code objects of the library (one offload bundle per source)."""
    fat = os.path.join(tmp, "fat")
    subprocess.run([OBJCOPY, "--dump-section", f".hip_fatbin={fat}", LIB, os.path.join(tmp, "copy.so")], check=True)
    data = open(fat, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n = struct.unpack_from("<Q", data, at + len(MAGIC))[0]
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def registers(text):
    """Vector registers named in an instruction's operands (not the accumulation half)."""
    regs = set()
    for a, b in re.findall(r"(?<![a-z0-9_])v\[(\d+):(\d+)\]", text):
        regs.update(range(int(a), int(b) + 1))
    regs.update(int(a) for a in re.findall(r"(?<![a-z0-9_])v(\d+)\b", text))
    return regs


def kernels(listing):
    """{name: [(address, mnemonic, operands, branch target or None)]}"""
    out, cur = {}, None
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if head:
            cur = out.setdefault(head.group(2), [])
            start = int(head.group(1), 16)
            continue
        ins = re.match(r"\s+([a-z]\w+)(.*?)\s*// ([0-9A-F]+):(?:.*<[^>]*?\+0x([0-9a-f]+)>)?", line)
        if ins and cur is not None:
            name, ops, addr, rel = ins.groups()
            target = start + int(rel, 16) if rel and name.startswith(("s_cbranch", "s_branch")) else None
            cur.append((int(addr, 16), name, ops, target))
    return out


def passes(name):
    """Passes (wait states) that a product holds the matrix core, 0 for other instructions."""
    return {"v_mfma_f32_32x32x16_bf16": 8, "v_mfma_f32_16x16x32_bf16": 4}.get(name, 0)


def too_early(code):
    """(product, offender) pairs within WAIT wait states, along every path.  An instruction
    takes one wait state, an s_nop its count and one, and a product waits until the matrix
    core is free of the one before."""
    index = {ins[0]: i for i, ins in enumerate(code)}
    bad, products = [], 0
    for i, (_, name, ops, _) in enumerate(code):
        if name != "v_mfma_f32_32x32x16_bf16":
            continue
        dst = ops.split(",")[0].strip()
        if not dst.startswith("v["):
            continue                       # a builtin's product, which the compiler tracks
        products += 1
        written = registers(dst)
        seen, work = {}, [(i + 1, 1, passes(name))]
        while work:
            j, now, free = work.pop()
            if j >= len(code) or any(n <= now and f <= free for n, f in seen.get(j, ())):
                continue
            seen.setdefault(j, []).append((now, free))
            _, nm, op, target = code[j]
            if passes(nm):
                now = max(now, free)
                free = now + passes(nm)
            if now > WAIT:
                continue
            if registers(op) & written:
                # the next product into the same registers is ordered by the matrix core
                if not (nm == name and op.split(",")[0].strip() == dst):
                    bad.append((f"{name} {ops.strip()}", f"{nm} {op.strip()} after {now - 1}"))
                    break
            if nm == "s_endpgm":
                continue
            now += int(op.strip(), 0) + 1 if nm == "s_nop" else 1
            if target is not None and target in index:
                work.append((index[target], now, free))
            if nm != "s_branch":
                work.append((j + 1, now, free))
    return products, bad


def test_the_walk_finds_an_early_use():
    mfma = (0, "v_mfma_f32_32x32x16_bf16", " v[0:15], v[32:35], a[0:3], 0", None)
    other = ("v_mfma_f32_32x32x16_bf16", " a[16:31], v[32:35], v[36:39], a[16:31]", None)
    end = (400, "s_endpgm", "", None)
    use = ("v_mul_f32_e32", " v40, v7, v41", None)
    assert too_early([mfma, (8, "s_nop", " 15", None), (12,) + use, end])[1]
    assert not too_early([mfma, (8, "s_nop", " 15", None), (12, "s_nop", " 1", None), (16,) + use, end])[1]
    # two products behind it hold the matrix core for 16 wait states
    assert not too_early([mfma, (8,) + other, (16,) + other, (24, "s_nop", " 1", None), (28,) + use, end])[1]
    assert too_early([mfma, (8,) + other, (16, "s_nop", " 0", None), (20,) + use, end])[1]
    # ... across a loop's back edge
    loop = [(0,) + use, mfma[:0] + (8,) + mfma[1:], (16, "s_cbranch_scc1", " 65000", 0), end]
    assert too_early(loop)[1]


@pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(OBJCOPY)), reason="no LLVM binary tools")
def test_no_instruction_touches_a_score_too_early(tmp_path):
    if not os.path.exists(LIB):
        pytest.fail("libheadcast.so is not built (run __graft_entry__.build())")
    found = {}
    for n, obj in enumerate(device_objects(str(tmp_path))):
        if b"attn_dense128_kernel" not in obj:
            continue
        path = tmp_path / f"{n}.o"
        path.write_bytes(obj)
        listing = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True).stdout
        found.update({k: v for k, v in kernels(listing).items() if "attn_dense128_kernel" in k})
    assert len(found) == 5, sorted(found)
    for name, code in found.items():
        products, bad = too_early(code)
        assert products >= 64, (name, products)
        assert not bad, (name, bad[:5])
