"""No loop of the device code runs a barrier or a cross-lane read while some of a wave's lanes have
left it: the compiler may turn a lane-dependent branch at the end of a loop into a loop of its own,
which those operations do not survive.  Read from the assembly of the kernels, on the CPU."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2505_17287_amd import build as B

CROSS_LANE = re.compile(r"s_barrier|ds_(bpermute|permute|swizzle)|.*\b(wave_sh|wave_ro|row_|quad_perm)")
# a wave works on one ghost: the trip counts are the same in every lane, which the compiler cannot know
UNIFORM = {"k_closest"}


def _kernels(text):
    name, body = None, []
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
        elif name and ".end_amdhsa_kernel" in line:
            yield name, body
            name = None
        elif name:
            body.append(line)


def _blocks(body):
    """Basic blocks as [label, instructions]."""
    out, cur = [], ["", []]

    def end():
        if cur[0] or cur[1]:
            out.append(cur)

    for line in body:
        line = line.split(";")[0].strip()
        m = re.match(r"(\.L\w+):", line)
        if m:
            end()
            cur = [m.group(1), []]
        elif line and not line.startswith("."):
            cur[1].append(line)
            if re.match(r"s_(cbranch|branch|endpgm)", line):
                end()
                cur = ["", []]
    end()
    return out


def split_loops(body):
    """(header, cross-lane operations) of the loops that lanes leave one by one: the block that ends
    a trip takes the lanes that are done out of exec."""
    blocks = _blocks(body)
    at = {b[0]: i for i, b in enumerate(blocks) if b[0]}
    pred = [[] for _ in blocks]
    for i, (_, code) in enumerate(blocks):
        last = code[-1] if code else ""
        m = re.match(r"s_c?branch\w*\s+(\.L\w+)", last)
        if m:
            pred[at[m.group(1)]].append(i)
        if not re.match(r"s_branch|s_endpgm", last) and i + 1 < len(blocks):
            pred[i + 1].append(i)
    found = []
    for i, (_, code) in enumerate(blocks):
        if not any(re.match(r"s_andn2_b64 exec, exec", c) for c in code):
            continue
        m = re.match(r"s_cbranch_exec(z|nz)\s+(\.L\w+)", code[-1])
        if not m:
            continue
        head = i + 1 if m.group(1) == "z" else at[m.group(2)]
        loop, todo = {head, i}, [i]
        while todo:
            j = todo.pop()
            for p in pred[j] if j != head else []:
                if p not in loop:
                    loop.add(p)
                    todo.append(p)
        ops = sorted({c.split()[0] for j in loop for c in blocks[j][1] if CROSS_LANE.match(c)})
        if ops:
            found.append((blocks[head][0], ops))
    return found


def test_the_check_sees_a_split_loop():
    whole = """
\ts_mov_b32 s0, 0
.LBB0_1:
\ts_barrier
\ts_and_saveexec_b64 s[2:3], vcc
\ts_cbranch_execz .LBB0_2
\tglobal_store_dword v0, v1, s[4:5]
.LBB0_2:
\ts_or_b64 exec, exec, s[2:3]
\ts_add_i32 s0, s0, 1
\ts_cmp_lt_i32 s0, s1
\ts_cbranch_scc1 .LBB0_1
.LBB0_3:
\tv_add_u32_e32 v2, 1, v2
\ts_andn2_b64 exec, exec, s[8:9]
\ts_cbranch_execnz .LBB0_3
\ts_barrier
\ts_endpgm
""".splitlines()
    assert split_loops(whole) == []
    split = [l.replace("s_cmp_lt_i32 s0, s1", "s_andn2_b64 exec, exec, s[6:7]").replace("scc1", "execnz") for l in whole]
    assert split_loops(split) == [(".LBB0_1", ["s_barrier"])]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")

    def one(src):
        path = str(out / (src + ".s"))
        r = subprocess.run([B.HIPCC, *B.FLAGS, "-S", "--offload-device-only", "-o", path, os.path.join(B.SRC, src)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(path).read()

    with ThreadPoolExecutor(max_workers=8) as ex:
        return dict(zip(B.SOURCES, ex.map(one, B.SOURCES)))


@pytest.mark.parametrize("src", [s for s in B.SOURCES if s != "api.hip"])
def test_no_loop_is_split_around_cross_lane_work(assembly, src):
    kernels = list(_kernels(assembly[src]))
    assert kernels
    bad = {n: l for n, l in ((n, split_loops(b)) for n, b in kernels) if l and not any(g in n for g in UNIFORM)}
    assert not bad
