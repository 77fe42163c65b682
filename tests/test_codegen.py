"""What the compiler makes of loops whose point is the order of their loads: a kernel is compiled for gfx950, by itself and with the
library's flags, and its assembly is read.  A source that asks for loads in flight together can compile to one round trip
after the other (a load behind a branch, or one merged into another) with every result still right, so that no other test sees it.
Needs hipcc, no GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1906_00091_amd import build as hip_build


def _assembly(tmp_path, include, kernels):
    src, out = str(tmp_path / "kernels.hip"), str(tmp_path / "kernels.s")
    with open(src, "w") as f:
        f.write('#include "%s"\nnamespace dlrm {\n%s\n}\n' % (include, "\n".join("template __global__ void %s;" % k for k in kernels)))
    cmd = [hip_build._hipcc()] + hip_build.HIPCC_FLAGS + ["--cuda-device-only", "-S", "-o", out, src]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("huge_run,builds", [(2048, True), (1024, False), (4096, False)])
def test_a_run_is_queued_or_reduced_in_its_bucket_but_never_both(tmp_path, huge_run, builds):
    """The limit from which a row split off an oversized bucket is queued has to be the size that the bucket's own reduction
    takes: with any other limit the sources must not compile."""
    csrc = str(tmp_path / "csrc")
    shutil.copytree(hip_build.CSRC, csrc)
    with open(os.path.join(csrc, "bwd_common.h")) as f:
        text, n = re.subn(r"constexpr int kHugeRun = \d+;", "constexpr int kHugeRun = %d;" % huge_run, f.read())
    assert n == 1
    with open(os.path.join(csrc, "bwd_common.h"), "w") as f:
        f.write(text)
    src = os.path.join(csrc, "one.hip")
    with open(src, "w") as f:
        f.write('#include "bwd_reduce.h"\nnamespace dlrm {\n'
                'template __global__ void bucket_reduce_kernel<DLRM_F32, 16, kSgd, false, false>(GroupArgs, UpdArgs);\n}\n')
    flags = ["-I" + csrc if f == hip_build.CSRC else f for f in hip_build.HIPCC_FLAGS if f != "-I"]
    flags = ["-I" + f if f == hip_build.INCLUDE else f for f in flags]
    r = subprocess.run([hip_build._hipcc()] + flags + ["--cuda-device-only", "-fsyntax-only", src], capture_output=True, text=True)
    assert (r.returncode == 0) == builds, r.stderr[-3000:]
    assert builds or "never both" in r.stderr, r.stderr[-3000:]


def _kernels(asm):
    """{kernel symbol: lines of its body}"""
    found, body = {}, None
    for line in asm.splitlines():
        t = line.strip()
        if re.match(r"_Z\w+:", t):
            body = found.setdefault(t.split(":")[0], [])
        elif t.startswith("s_endpgm"):
            body = None
        elif body is not None and t and not t.startswith(";"):
            body.append(t)
    return found


def _waits_for_loads(t):
    return t.startswith("s_waitcnt") and "vmcnt" in t


def _longest_run(lines, load):
    """Most loads that match with no wait for a load, no branch and no label among them."""
    best = run = 0
    for t in lines:
        if re.match(load, t):
            run += 1
            best = max(best, run)
        elif _waits_for_loads(t) or t.startswith(("s_cbranch", "s_branch", ".LBB")):
            run = 0
    return best


def test_weighted_entries_of_a_bucket_are_requested_together(tmp_path):
    """A sorted bucket's (bag, weight) records, 8 bytes each and up to 8 a thread (fp32 rows: no other load of 8 bytes comes
    more than a few at a time)."""
    asm = _assembly(tmp_path, "bwd_reduce.h", ["bucket_reduce_kernel<DLRM_F32, 16, %s, true, false>(GroupArgs, UpdArgs)" % o
                                               for o in ("kSgd", "kAdagrad")])
    bodies = _kernels(asm)
    assert len(bodies) == 2
    for name, lines in bodies.items():
        assert _longest_run(lines, r"(global|flat)_load_dwordx2 ") >= 8, name


def _loads_behind_rows(lines, row, index, rows):
    """True if an `index` load follows `rows` loads of rows that have not been waited for, in one pass over straight code."""
    pending = 0
    for t in lines:
        if re.match(row, t):
            pending += 1
        elif re.match(index, t) and pending >= rows:
            return True
        elif t.startswith(".LBB") or (_waits_for_loads(t) and pending >= rows and
                                      int(re.search(r"vmcnt\((\d+)\)", t).group(1)) < rows):
            pending = 0
    return False


def test_pooling_requests_the_next_indices_behind_this_round_s_rows(tmp_path):
    """A lane group per bag: four rows are requested, then the next round's indices, before anything is waited for."""
    asm = _assembly(tmp_path, "emb_fwd.hip", [])
    bodies = {n: b for n, b in _kernels(asm).items() if "emb_fwd_group_kernel" in n}
    assert len(bodies) == 3 * 7 * 2 * 2   # storage types, lanes per row, weights, index types
    for name, lines in bodies.items():
        index = r"global_load_dword " if "EiEEv" in name else r"global_load_dword(x2)? "
        assert _loads_behind_rows(lines, r"global_load_dwordx4 ", index, 4), name


def _rows_in_flight(lines, row):
    """Of every straight piece of code with loads that match: how many there are, and how many are on their way at once."""
    found, total, flying, most = [], 0, 0, 0
    for t in lines + [".LBB"]:
        if t.startswith(("s_cbranch", "s_branch", ".LBB")):
            if total:
                found.append((total, most))
            total = flying = most = 0
        elif re.match(row, t):
            total, flying = total + 1, flying + 1
            most = max(most, flying)
        elif _waits_for_loads(t):   # loads return in order: a wait that leaves n on their way may be for an older one
            flying = min(flying, int(re.search(r"vmcnt\((\d+)\)", t).group(1)))
    return found


def test_pooling_by_wavefronts_requests_the_rows_of_a_round_together(tmp_path):
    """A wavefront per bag, alone or walking several: 16-bit rows of a round, of eight or of a bag's last rounds, are all requested
    before one is waited for (64 positions are at most G rounds of 64 / G rows; rows of 64 lanes are pooled by lane groups);
    where the compiler is left to itself, with fp32 rows, more than half of them."""
    asm = _assembly(tmp_path, "emb_fwd.hip", [])
    bodies = {n: b for n, b in _kernels(asm).items() if re.search(r"emb_fwd_wave(_seq)?_kernel", n)}
    assert len(bodies) == 2 * 3 * 7 * 2 * 2   # kernels, storage types, lanes per row, weights, index types
    for name, lines in bodies.items():
        dtype, lanes = (int(x) for x in re.search(r"ILi(\d)ELi(\d+)ELi8E", name).groups())
        if lanes == 64:
            continue
        rounds = _rows_in_flight(lines, r"global_load_dwordx4 ")
        assert all(total == most if dtype else 2 * most > total for total, most in rounds), (name, rounds)
        assert max(total for total, _ in rounds) >= min(8, lanes), (name, rounds)


def _occupancy(asm):
    """{kernel symbol: wavefronts per SIMD that its registers allow}"""
    return _figures(asm, "Occupancy")


def _figures(asm, which):
    """{kernel symbol: one of the figures that the compiler states behind it}"""
    found, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        name = m.group(1) if m else name
        m = re.match(r"; %s: (\d+)" % which, line)
        if m:
            found[name] = int(m.group(1))
    return found


def test_one_launch_forward_of_33_to_48_tables_keeps_four_wavefronts_per_simd(tmp_path):
    """Its registers are just below the limit for four; with the dense row held through the products they are above it."""
    found = {n: o for n, o in _occupancy(_assembly(tmp_path, "pooled_interact.hip", [])).items() if "pooled_interact_fwd_kernelILi3E" in n}
    assert len(found) == 3 * 2   # storage types, index types
    assert min(found.values()) >= 4, found


def test_interaction_forward_keeps_its_tiles_in_registers(tmp_path):
    """No row block count spills: staged rows wait in registers while the columns before them are multiplied."""
    asm = _assembly(tmp_path, "interact.hip", [])
    found = {n: v for n, v in _figures(asm, "ScratchSize").items() if "interact_fwd" in n}
    assert len(found) == 7 + 7 and not any(found.values()), found   # a wavefront per sample, several
    narrow = [v for n, v in _occupancy(asm).items() if "interact_fwd_split_kernelILi8ELi4ELb0E" in n]   # no staged rows wait there
    assert len(narrow) == 1 and narrow[0] >= 4, narrow   # workgroups that fit the LDS


def test_sums_of_narrow_rows_read_several_pieces_of_a_run_together(tmp_path):
    """A run over many slabs of a bucket: up to 255 of them with rows of 4 columns.  Eight pieces (16 bytes of LDS a lane) are
    requested before one is waited for; the compiler puts a branch before the last of them."""
    which = [("DLRM_F32", 1, "kSgd", "false"), ("DLRM_F32", 4, "kAdagrad", "true"), ("DLRM_F16", 2, "kSgd", "false"),
             ("DLRM_BF16", 8, "kAdagrad", "false")]
    asm = _assembly(tmp_path, "bwd_reduce.h", ["bucket_reduce_kernel<%s, %d, %s, %s, false>(GroupArgs, UpdArgs)" % w for w in which])
    bodies = _kernels(asm)
    assert len(bodies) == len(which)
    for name, lines in bodies.items():
        best = run = 0
        for t in lines:
            if t.startswith("ds_read_b128 "):
                run += 1
                best = max(best, run)
            elif (t.startswith("s_waitcnt") and "lgkmcnt" in t) or t.startswith(("s_cbranch", "s_branch", ".LBB")):
                run = 0
        assert best >= 7, (name, best)
