"""The listing of the library's kernels: no vector-memory instruction reads a scalar register within the five wait states that it has
to stay behind the vector unit's writing it.  The compiler keeps that distance between instructions of its own; requests written
in assembly blocks it does not look into."""
import collections
import re
import struct
import subprocess

import pytest

from paper_2512_17452_amd.binding import library_path

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 5


def _code_objects(data):
    """The GPU code objects in the fat binary of a library: magic, number of entries, (offset, size, length of the name, name) each."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + ln]
            p += 24 + ln
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


def _scalars(token):
    m = re.match(r"s\[(\d+):(\d+)\]", token)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"s(\d+)$", token)
    return {int(m[1])} if m else {"vcc"} if token.startswith("vcc") else set()


def _too_close(listing):
    """(kernel, writer, reader, wait states) of every pair that is too close, along every way through the kernel's branches."""
    found = []

    def check(name, ins):
        index = {addr: i for i, (addr, _, _) in enumerate(ins)}
        before = collections.defaultdict(list)
        for i, (addr, op, args) in enumerate(ins):
            if op.startswith("s_cbranch") or op == "s_branch":
                off = int(args[0])
                to = index.get(addr + 4 + 4 * (off - 65536 if off > 32767 else off))
                if to is not None:
                    before[to].append(i)
            if i + 1 < len(ins) and op not in ("s_branch", "s_endpgm"):
                before[i + 1].append(i)
        for i, (addr, op, args) in enumerate(ins):
            if not re.match(r"(global|buffer|flat|scratch)_", op):
                continue
            reads = set().union(*map(_scalars, args))
            seen, todo = {}, [(i, 0)] if reads else []
            while todo:
                j, waited = todo.pop()
                for k in before[j]:
                    _, kop, kargs = ins[k]
                    if kop.startswith("v_") and kargs and any(_scalars(x) & reads for x in kargs[:2 if "_co_" in kop else 1]):
                        found.append((name, " ".join([kop] + kargs), " ".join([op] + args), waited))
                        continue
                    w = waited + (int(kargs[0]) + 1 if kop == "s_nop" else 1)
                    if w < WAIT_STATES and seen.get(k, WAIT_STATES) > w:
                        seen[k] = w
                        todo.append((k, w))

    name, ins = None, []
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            check(name, ins)
            name, ins = m[1], []
            continue
        m = re.match(r"\s+(\S+)(.*?)//\s*([0-9A-F]+):", line)
        if m:
            ins.append((int(m[3], 16), m[1], [x.split()[0] for x in m[2].split(",") if x.split()]))
    check(name, ins)
    return found


def test_the_check_itself():
    line = "\t%s // %012X: 00\n"
    near = ["v_readlane_b32 s5, v1, s2", "s_mov_b32 m0, s9", "s_nop 0", "global_load_lds_dwordx4 v3, s[4:5] nt"]
    far = near[:2] + ["s_nop 3"] + near[3:]
    copied = near[:2] + ["s_mov_b64 s[6:7], s[4:5]", "global_load_lds_dwordx4 v3, s[6:7] nt"]
    around = ["global_load_lds_dwordx4 v3, s[4:5] nt", "v_readlane_b32 s5, v1, s2", "s_cbranch_scc1 65533"]
    for code, want in ((near, 1), (far, 0), (copied, 0), (around, 1)):
        text = "0000 <k>:\n" + "".join(line % (c, 4 * i) for i, c in enumerate(code))
        assert len(_too_close(text)) == want, code


def test_vector_writes_of_scalars_stay_ahead_of_requests(tmp_path):
    try:
        data = open(library_path(), "rb").read()
    except FileNotFoundError:
        pytest.skip("the library has not been built")
    n_requests = 0
    for i, code in enumerate(_code_objects(data)):
        f = tmp_path / f"{i}.co"
        f.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", str(f)], capture_output=True, text=True, check=True).stdout
        n_requests += listing.count("global_load_lds_dwordx4")
        found = _too_close(listing)
        assert not found, (len(found), found[:5])
    assert n_requests > 0
