"""What the compiler made of the kernels: properties of the gfx950 code in libsdconv.so that the sources rely on
and no result shows reliably."""
import heapq
import os
import re
import shutil
import subprocess

import pytest

import paper_1903_05831_amd as sd
from paper_1903_05831_amd import build, fit_models

LLVM = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin")
LINE = re.compile(r"^\t(\S+)(.*?)\s*// ([0-9A-F]+):.*?(?:<(\S+?)(?:\+0x([0-9a-fA-F]+))?>)?$")
NONE = 99       # no LDS read on its way


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    where = tmp_path_factory.mktemp("code")
    sd.lib()
    shutil.copy(build.LIB, where / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=where, check=True, capture_output=True)
    out = sorted(str(p) for p in where.iterdir() if p.name.endswith("gfx950"))
    assert len(out) > 10, out
    return out


def _kernels(path):
    """(name, [(address, instruction, operands, address it may jump to)]) of every function."""
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", path], check=True, capture_output=True, text=True).stdout
    name, start, body = None, 0, []
    for line in text.splitlines():
        if head := re.match(r"^([0-9a-f]+) <(\S+)>:$", line):
            if name:
                yield name, body
            start, name, body = int(head[1], 16), head[2], []
        elif m := LINE.match(line):
            target = None
            if m[4] is not None:
                target = start + int(m[5] or "0", 16) if m[4] == name else None
                assert target is not None, (path, line)
            body.append((int(m[3], 16), m[1], m[2], target))
    if name:
        yield name, body


def _reads_at_barriers(body):
    """Addresses of the barriers that a wave can reach with one of its LDS reads on its way.

    Carried along every path: how many LDS operations the wave has issued after its last read (they complete
    in order, so lgkmcnt(n) has waited for that read if n is no more than this), or NONE."""
    at = {a: i for i, (a, _, _, _) in enumerate(body)}
    state, todo, found = {0: NONE}, [0], set()
    while todo:
        i = todo.pop()
        after, (addr, op, args, target) = state[i], body[i]
        if op == "s_barrier" and after != NONE:
            found.add(addr)
        if op.startswith("ds_"):
            after = 0 if "read" in op else min(after + 1, 15) if after != NONE else NONE
        elif op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", args)
            n = int(m[1]) if m else 0 if args.strip() == "0" else 15
            if n <= after:
                after = NONE
        nexts = [] if op in ("s_endpgm", "s_branch", "s_setpc_b64") else [i + 1]
        if target is not None:
            nexts.append(at[target])
        for n in nexts:
            if n < len(body) and after < state.get(n, NONE + 1):
                state[n] = after
                todo.append(n)
    return found


def test_barriers_of_lds_dma_kernels_are_reached_with_no_lds_read_on_its_way(code_objects):
    """Behind a barrier an LDS-DMA load of another wave may overwrite what was read before it, and s_barrier itself
    waits for nothing: a wave must have its values by then, on every path through the code."""
    bad, kernels = [], 0
    for path in code_objects:
        for name, body in _kernels(path):
            if any(op.startswith("buffer_load") and args.endswith(" lds") for _, op, args, _ in body):
                kernels += any(op == "s_barrier" for _, op, _, _ in body)
                bad += [(name, hex(a)) for a in _reads_at_barriers(body)]
    assert kernels > 40
    assert not bad, bad


def _notes(path):
    """Fields of every kernel's metadata."""
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, capture_output=True, text=True).stdout
    return [{k: v for k, v in re.findall(r"\.(\w+):\s+(\S+)", kernel)} for kernel in notes.split("- .agpr_count")[1:]]


def test_no_kernel_spills_registers_or_uses_scratch_memory(code_objects):
    kernels = 0
    for path in code_objects:
        for field in _notes(path):
            assert field["vgpr_spill_count"] == "0" and field["private_segment_fixed_size"] == "0", (field["name"], field)
            kernels += 1
    assert kernels > 100


def test_a_plain_stem_call_does_not_carry_the_registers_of_a_tail(code_objects):
    """The stem's forward kernel without a tail, with the one in LDS and with any: one kernel for all made plain calls 5 % slower
    than they were without the second."""
    found = {m[1]: field for path in code_objects for field in _notes(path)
             if (m := re.search(r"thin_fwd_kernel(?:ILi(\d)E)?", field["name"]))}
    assert sorted(found) == ["0", "1", "2"], found.keys()
    vector, scalar = ({k: int(f[name]) for k, f in found.items()} for name in ("vgpr_count", "sgpr_spill_count"))
    assert vector["0"] < min(vector["1"], vector["2"]), vector
    assert scalar["0"] < 20 and scalar["1"] < 20, scalar       # 90 in the one kernel


def test_workgroups_that_are_to_share_a_compute_unit_have_the_registers_for_it(code_objects):
    """The time models count on so many workgroups of some tiles on a compute unit, with a tail or without: four SIMDs of 512
    registers, taken in eights."""
    tiles = {(128, 128, 2): 2, (128, 64, 2): 3, (64, 64, 4): 2}       # height, width, stages of the ring: fit_models.PER_CU 339, 340, 327 and 328
    found = set()
    for path in code_objects:
        for field in _notes(path):
            m = re.match(r"_ZN6sdconv15igemm_ws_kernelILi\dELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi64ELi(\d+)E", field["name"])
            if m and (tile := (int(m[1]), int(m[2]), int(m[5]))) in tiles:
                waves = (int(m[3]) * int(m[4]) + int(m[6])) * tiles[tile] // 4
                assert -(-int(field["vgpr_count"]) // 8) * 8 * waves <= 512, (field["name"], field["vgpr_count"], waves)
                found.add((tile, field["name"]))
    assert len(found) == 16, found      # two passes, plain and with a tail; two kinds of 64x64


def _trips_to_the_first_load(body):
    """Waits for kernel parameters in lines of 64 bytes not read before, on the way to the first LDS-DMA load that has the fewest."""
    at = {a: i for i, (a, _, _, _) in enumerate(body)}
    heap, seen = [(0, 0, (), ())], set()
    while heap:
        trips, i, read, asked = heapq.heappop(heap)
        if (i, read, asked) in seen:
            continue
        seen.add((i, read, asked))
        _, op, args, target = body[i]
        if op.startswith("buffer_load") and args.endswith(" lds"):
            return trips
        if op.startswith("s_load"):
            m = re.match(r"\s*\S+, (s\[\d+:\d+\]), (0x[0-9a-f]+|\d+)", args)
            first, size = int(m[2], 0), 4 * int(re.sub(r"\D", "", op) or "1")
            asked = tuple(sorted({*asked, *((m[1] == "s[0:1]", line) for line in (first // 64, (first + size - 1) // 64))} - set(read)))
        elif op == "s_waitcnt" and "lgkmcnt(0)" in args and asked:
            trips, read, asked = trips + 1, tuple(sorted({*read, *asked})), ()
        for n in ([] if op in ("s_endpgm", "s_branch", "s_setpc_b64") else [i + 1]) + ([] if target is None else [at[target]]):
            if n < len(body):
                heapq.heappush(heap, (trips, n, read, asked))


def test_kernels_ask_for_their_parameters_at_once(code_objects):
    """Left to the compiler, the split-role kernels waited for parameters in two to five cold lines, one after the other, before
    their first operand load, and a change of code far from there could add one."""
    trips = {name: _trips_to_the_first_load(body) for path in code_objects for name, body in _kernels(path)
             if re.match(r"_ZN6sdconv19igemm_ws_f32_kernel|_ZN6sdconv15igemm_ws_kernel", name)}
    assert len(trips) > 80 and all(n <= (3 if "f32" in name else 2) for name, n in trips.items()), trips


def test_the_library_holds_the_variants_that_can_be_chosen(monkeypatch):
    """Those of the time models and of the rule for large tensors (0, 3; 0, 1), and no others."""
    d, known = sd.make_desc(1, 28, 28, 64, 64, 3, 3, (1, 1), (1, 1)), set()
    for env, variants, passes in (("SDCONV_IGEMM_VARIANT", [0, 3] + fit_models.ROW_VARIANTS, (sd.FWD, sd.DGRAD)),
                                  ("SDCONV_WGRAD_VARIANT", [0, 1] + fit_models.WGRAD_MODELS, (sd.WGRAD,))):
        for v in variants:
            monkeypatch.setenv(env, str(v))
            known |= {sd.kernel_name(d, p) for p in passes}
        monkeypatch.delenv(env)
    with open(build.LIB, "rb") as f:
        names = re.findall(rb"(?<=\0)((?:igemm_(?:fwd|dgrad)|conv_(?:fwd|dgrad)_patch|wgrad(?:_dma)?)_[a-z0-9_]*\d+x\d+[a-z0-9_]*)(?=\0)", f.read())
    assert {n.decode() for n in names} == known
