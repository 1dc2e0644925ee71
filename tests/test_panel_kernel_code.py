"""The panel kernel's generated code (gemm_mid.hip), no GPU: its requests to memory go to LDS behind counted waits, which hold only if
the compiler keeps the requests in the order they are written in, and a register that is kept in scratch memory is a request more among
them.  The compiled assembly is walked along every path with the requests in flight: when LDS is read, no activations may be on their way
there, and codes only as many as an odd group leaves (2 per tile of channels)."""
import re
import subprocess

import pytest

from paper_2410_08661_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "gemm_mid.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-w", "--cuda-device-only", "-S", f"{build.CSRC}/gemm_mid.hip", "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def _kernels(text):
    for m in re.finditer(r"^(_ZN\S*fwd_mid_kernelILi(\d)ELi(\d)ELNS0_3FmtE(\d)\S*):.*?^\.Lfunc_end", text, re.M | re.S):
        code, labels = [], {}
        for line in m.group(0).splitlines()[1:]:
            line = line.split(";")[0].strip()
            label = re.match(r"(\.LBB\S+):", line)
            if label:
                labels[label.group(1)] = len(code)
            elif line and not line.startswith("."):
                code.append(line)
        yield m.group(1), int(m.group(3)), int(m.group(4)), code, labels


def _in_flight_at_reads(code, labels):
    """Sets of (descriptor, requests) on their way to LDS when an LDS read is issued, over all paths."""
    found, seen, work = set(), set(), [(0, ())]
    while work:
        pc, queue = work.pop()
        while True:
            op, _, args = code[pc].partition(" ")
            if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
                queue = (*queue[-62:], re.search(r"s\[\d+:\d+\]", args).group(0) if args.endswith(" lds") else "")   # (no wait leaves more than 63)
            elif op == "s_waitcnt":
                count = re.search(r"vmcnt\((\d+)\)", args)
                if count:
                    queue = queue[max(0, len(queue) - int(count.group(1))):]
            elif op.startswith("ds_read"):
                to_lds = [q for q in queue if q]
                if to_lds:
                    found.add((tuple(sorted(set(to_lds))), len(to_lds)))
            elif op == "s_endpgm":
                break
            if op == "s_branch" or op.startswith("s_cbranch"):
                at = (labels[args], queue)
                if at not in seen:
                    seen.add(at)
                    work.append(at)
                if op == "s_branch" or (pc + 1, queue) in seen:
                    break
                seen.add((pc + 1, queue))
            pc += 1
    return found


def test_no_request_to_lds_is_read_early(assembly):
    kernels = list(_kernels(assembly))
    assert len(kernels) == 60
    for name, nt, fmt, code, labels in kernels:
        found = _in_flight_at_reads(code, labels)
        if fmt == 0:      # 4-bit: the next pair's codes alone, one descriptor
            assert len(found) == 1 and all(len(d) == 1 and n == 2 * nt for d, n in found), (name, found)
        else:
            assert not found, (name, found)


def test_no_register_goes_to_scratch_memory(assembly):
    spilled = re.findall(r"\.symbol:\s+(\S*fwd_mid_kernel\S*).*?\.vgpr_spill_count:\s+(\d+)", assembly, re.S)
    assert len(spilled) == 60 and all(n == "0" for _, n in spilled), [s for s in spilled if s[1] != "0"]
