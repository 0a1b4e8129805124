"""What the compiled kernels have to hold whatever the compiler makes of the source: read from the disassembly of the
built library's own gfx950 code (no GPU needed)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP, READELF = "/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    """name -> (address, instruction, address it branches to or None), in the order of the code."""
    from paper_2506_03887_amd.binding import LIB_PATH
    at = tmp_path_factory.mktemp("code")
    shutil.copy(LIB_PATH, at / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(at / "lib.so")], check=True, capture_output=True)
    out = {}
    for f in glob.glob(str(at / "lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
            if m:
                begin, name = int(m.group(1), 16), m.group(2)
                out[name] = []
                continue
            # instruction // address: code words <kernel+0xoffset of a branch's target>
            m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):[ 0-9A-F]*(?:<[^+>]+(?:\+0x([0-9a-f]+))?>)?$", line)
            if name and m:
                target = begin + int(m.group(3) or "0", 16) if "<" in line else None
                out[name].append((int(m.group(2), 16), m.group(1), target))
    assert out
    return out


@pytest.fixture(scope="module")
def spilled_scalars(tmp_path_factory):
    """name -> scalar registers kept in lanes of vector registers, by the code object's own notes."""
    from paper_2506_03887_amd.binding import LIB_PATH
    at = tmp_path_factory.mktemp("notes")
    shutil.copy(LIB_PATH, at / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(at / "lib.so")], check=True, capture_output=True)
    text = "".join(subprocess.run([READELF, "--notes", f], check=True, capture_output=True, text=True).stdout
                   for f in glob.glob(str(at / "lib.so.*gfx950")))
    names, counts = re.findall(r"^ {4}\.name: +(\S+)$", text, re.M), re.findall(r"^ {4}\.sgpr_spill_count: +(\d+)$", text, re.M)
    assert names and len(names) == len(counts)
    return dict(zip(names, map(int, counts)))


@pytest.fixture(scope="module")
def kernels(listing):
    """name -> instructions, in the order of the code."""
    return {name: [text for _, text, _ in code] for name, code in listing.items()}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_a_block_of_the_spread_step_counts_itself_in_when_its_loads_have_returned(kernels):
    """The blocks of a row read its stack, count themselves in, and the last to do so overwrites the stack: between the
    last load before the count (the first atomic that returns a value) and the count, the wave has to wait for all loads."""
    found = {n: code for n, code in kernels.items() if "step_spread_kernel" in n}
    assert len(found) == 4
    for name, code in found.items():
        count = next(i for i, x in enumerate(code) if re.match(r"global_atomic_add\b.*\bsc0\b", x))
        loads = [i for i, x in enumerate(code[:count]) if re.match(r"(global|flat|buffer|scratch)_load", x)]
        waits = [i for i, x in enumerate(code[:count]) if re.match(r"s_waitcnt\b.*vmcnt\(0\)", x)]
        assert waits and waits[-1] > loads[-1], name
        between = [x for x in code[waits[-1]: count] if re.match(r"s_cbranch|s_branch", x)]
        assert all(x.startswith("s_cbranch_execz") for x in between), (name, between)     # straight code, lanes switched off at most


def _registers(operand):
    """The registers an operand names: s3, v[4:7], vcc, ..."""
    m = re.match(r"^[-|]*([sva])\[(\d+):(\d+)\]|^[-|]*([sva])(\d+)\b", operand)
    if not m:
        return ["vcc"] if operand.startswith("vcc") else []
    if m.group(1):
        return [m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)]
    return [m.group(4) + m.group(5)]


class _Inputs:
    """Which registers (and lanes that spilled scalars sit in) hold addresses of tokens, len or states -- the first 24 bytes of the
    arguments, in s[2:7] when the kernel starts --, and which of their loads are still out, at every instruction of a kernel:
    a forward data flow over its branches, joined by union.  Addresses are moved, spilled and added to; other arithmetic on
    what may hold one makes none."""
    ADDRESS = re.compile(r"s_mov_b(32|64)|s_addc?_u32|s_cselect_b(32|64)|v_mov_b(32|64)|v_lshl_add_u64|v_addc?_co_u32|v_cndmask|v_read|s_or_b32|v_or_b32")
    NO_RESULT = re.compile(r"(s_cmp|s_bitcmp|s_cbranch|s_branch|s_waitcnt|s_barrier|s_nop|s_endpgm|s_setprio|s_sleep|global_store|flat_store|"
                           r"buffer_store|ds_write|s_dcache|buffer_|v_cmpx)")

    def __init__(self, code):
        self.code, self.at = code, {address: i for i, (address, _, _) in enumerate(code)}
        self.seen = [None] * len(code)
        self.loads = set()
        self.run(0, frozenset("s%d" % i for i in range(2, 8)))

    def run(self, start, state):
        todo = [(start, state)]
        while todo:
            i, state = todo.pop()
            if self.seen[i] is not None:
                if state <= self.seen[i]:
                    continue
                state |= self.seen[i]
            self.seen[i] = state
            out = self.step(i, state)
            todo += [(n, out) for n in self.follow(i)]

    def follow(self, i):
        _, text, target = self.code[i]
        if text.startswith("s_endpgm"):
            return []
        assert not re.match(r"s_(setpc|swappc|call)", text), text
        next_ = [] if text.startswith("s_branch") else [i + 1]
        return next_ + ([self.at[target]] if re.match(r"s_c?branch", text) else [])

    def step(self, i, state):
        text = self.code[i][1]
        name, _, rest = text.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if name == "s_waitcnt":
            return frozenset(x for x in state if not ((x == "scalar out" and "lgkmcnt(0)" in text) or (x == "vector out" and "vmcnt(0)" in text)))
        if self.NO_RESULT.match(name) or not rest:
            return state
        results = 2 if re.match(r"v_\w+_co_\w+|v_div_scale|v_mad_[iu]64", name) else 1                  # (a carry)
        made, used = [r for o in ops[:results] for r in _registers(o)], [r for o in ops[results:] for r in _registers(o)]
        if name == "v_writelane_b32":
            slot = "%s.%s" % (ops[0], ops[2])
            return state | {slot} if made and _registers(ops[1])[:1] and _registers(ops[1])[0] in state else state - {slot}
        if name == "v_readlane_b32" and ops[2].isdigit():
            tainted = "%s.%s" % (ops[1], ops[2]) in state
            return state | set(made) if tainted else state - set(made)
        if re.match(r"(s_|s_buffer_|global_|flat_|buffer_|scratch_|ds_)(load|read)", name):
            state -= set(made)
            if name.startswith("s_load") and _registers(ops[1]) == ["s0", "s1"] and i < self.entry():
                first = int(ops[2].split()[0], 16)                          # the arguments themselves
                return state | {r for k, r in enumerate(made) if first + 4 * k < 24}
            if any(r in self.seen[i] for r in used):
                self.loads.add(i)
                return state | {"scalar out" if name.startswith("s_") else "vector out"}
            return state
        if re.match(r"(global|flat|buffer)_", name):                            # an atomic
            return state - set(made) if "sc0" in text else state
        address = self.ADDRESS.match(name) and any(r in state for r in used)
        return state | set(made) if address else state - set(made)

    def entry(self):
        """Up to here s[0:1] is the address of the arguments: its first change."""
        if not hasattr(self, "_entry"):
            changes = [i for i, (_, t, _) in enumerate(self.code) if not self.NO_RESULT.match(t) and
                       set(_registers(t.partition(" ")[2].split(",")[0].strip())) & {"s0", "s1"}]
            self._entry = min(changes, default=len(self.code))
        return self._entry

    def reachable(self, i):
        out, todo = set(), list(self.follow(i))
        while todo:
            n = todo.pop()
            if n not in out:
                out.add(n)
                todo += self.follow(n)
        return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_a_block_of_the_spread_step_has_read_its_inputs_when_it_counts_itself_in(listing):
    """tokens, len and states come through scalar loads, which no fence orders, and the last block overwrites them: each is
    loaded once, has returned before the count (the first atomic that returns a value), and is not loaded behind it."""
    found = {n: code for n, code in listing.items() if "step_spread_kernel" in n}
    assert len(found) == 4
    for name, code in found.items():
        flow = _Inputs(code)
        count = next(i for i, (_, x, _) in enumerate(code) if re.match(r"global_atomic_add\b.*\bsc0\b", x))
        assert flow.seen[count] is not None and len(flow.loads) == 3, (name, [code[i] for i in flow.loads])
        assert not flow.seen[count] & {"scalar out", "vector out"}, name
        assert not flow.loads & flow.reachable(count), name


def test_the_flow_of_input_addresses_sees_a_late_load():
    """The analysis on a few lines: an address spilled to a lane and used behind the count, and a load not waited for."""
    def flow(*lines):
        code = [(4 * i, x, None) for i, x in enumerate(lines)]
        branches = [(4 * i, x, 4 * int(x.split()[1])) if x.startswith("s_cbranch") else (4 * i, x, None) for i, x in enumerate(lines)]
        return _Inputs(branches if any(b[2] for b in branches) else code)
    early = ("s_add_u32 s8, s2, s12", "s_addc_u32 s9, s3, s13", "s_load_dword s20, s[8:9], 0x0", "s_waitcnt lgkmcnt(0)")
    count = "global_atomic_add v1, v2, v3, s[10:11] sc0"
    f = flow(*early, count, "s_endpgm")
    assert f.loads == {2} and "scalar out" not in f.seen[4]
    assert "scalar out" in flow(*early[:3], count, "s_endpgm").seen[3]
    f = flow("v_writelane_b32 v9, s6, 1", "s_mov_b32 s6, 0", "v_writelane_b32 v9, s7, 2", count, "v_readlane_b32 s30, v9, 1",
             "v_readlane_b32 s31, v9, 2", "s_load_dword s20, s[30:31], 0x0", "s_endpgm")
    assert f.loads == {6} and 6 in f.reachable(3)
    f = flow("s_cbranch_scc1 3", "s_mov_b64 s[4:5], 0", "s_nop 0", "s_load_dword s20, s[4:5], 0x0", "s_endpgm")     # tainted on one way
    assert f.loads == {3}
    assert flow("s_mov_b64 s[4:5], 0", "s_load_dword s20, s[4:5], 0x0", "s_endpgm").loads == set()


def test_lanes_exchange_words_through_lds_behind_a_fence():
    """What a lane lays in LDS for other lanes of its wave is read behind wave_exchange, whose fences hold the compiler (the wave
    barrier alone does not), and as the words or bytes it was written as: a read through a pointer to 16-bit values need
    not see stores of words."""
    from paper_2506_03887_amd.build import CSRC
    text = {os.path.basename(f): open(f).read() for f in glob.glob(os.path.join(CSRC, "*.h*"))}
    assert {f: t.count("__builtin_amdgcn_wave_barrier") for f, t in text.items() if "__builtin_amdgcn_wave_barrier" in t} == {"argmax.hpp": 1}
    fenced = r"ATOMIC_RELEASE, \"wavefront\", \"local\"\);\s+__builtin_amdgcn_wave_barrier\(\);\s+\S+ATOMIC_ACQUIRE, \"wavefront\", \"local\""
    assert re.search(fenced, text["argmax.hpp"])
    assert text["advance_kernels.hip"].count("wave_exchange()") >= 7 and "reinterpret_cast<const int16_t *>(s" not in text["advance_kernels.hip"]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_which_steps_look_for_the_plan_by_themselves(kernels):
    """The waves of the greedy step poll for the plan where the row's logits take longer than the advance (ten to seventeen groups
    per lane); shorter rows, which lose by it, the longest and every other form meet at a barrier."""
    polls = {n for n, code in kernels.items() if "advance_fill_apply_kernel" in n and any(x.startswith("s_sleep") for x in code)}
    assert {re.search(r"kernelILb[01]ELi(\d+)ELb(\d)ELi(\d)E", n).groups() for n in polls} == {("17", "1", "1")} and len(polls) == 2


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_scalars_that_the_greedy_step_of_two_rows_keeps_in_lanes(spilled_scalars):
    """Half the registers of a unit for each of two blocks: no more scalars in lanes than the form was measured with (231; the window
    and the token's line in flight together took 368)."""
    found = {n: c for n, c in spilled_scalars.items() if re.search(r"advance_fill_apply_kernelILb[01]ELi\d+ELb1ELi2E", n)}
    assert len(found) == 2 and max(found.values()) <= 231, found
