"""Properties of the built kernels that the sources cannot state, read from the library's own gfx950 code objects."""
import os
import re
import subprocess

import pytest

from paper_2511_11641_amd import build as bld

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The device code objects inside the library, one file per translation unit."""
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no LLVM tools")
    if not os.path.exists(bld.LIB):
        bld.build(verbose=False)
    d = tmp_path_factory.mktemp("co")
    os.symlink(bld.LIB, d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    files = sorted(str(d / f) for f in os.listdir(d) if "gfx950" in f)
    assert files
    return files


def test_no_scratch_memory(code_objects):
    """Every kernel of a pass keeps its values in registers (spills would travel beside the direct loads of the main loops)."""
    scratch = {}
    for f in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f], check=True, capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, flags=re.S):
            scratch[name] = int(size)
    assert len(scratch) > 100
    assert {n: s for n, s in scratch.items() if s and "mfma_probe" not in n} == {}


# ---- inline assembly -------------------------------------------------------------------------------------------------------------------
# The kernels that read LDS through inline assembly wait for those reads themselves, in another statement: the compiler takes a result as
# written at once and would be free to copy, spill or reuse its register while the read is under way.  Nor does it count wait states for
# matrix instructions written as assembly.  Both are checked on what it made of them.
REG = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])(?![\w])")


def _regs(text):
    out = set()
    for m in REG.finditer(text):
        out.update((m[1], i) for i in (range(int(m[2]), int(m[2]) + 1) if m[2] else range(int(m[3]), int(m[4]) + 1)))
    return out


def _functions(code_object):
    """{name: [(address, mnemonic, operands, branch target or None)]}"""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", code_object], check=True, capture_output=True, text=True).stdout
    funcs, cur, base = {}, None, 0
    for line in text.splitlines():
        if m := re.match(r"^([0-9a-f]+) <(.+)>:", line):
            base, cur = int(m[1], 16), funcs.setdefault(m[2], [])
        elif cur is not None and (m := re.match(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-Fa-f]+):(.*)$", line)):
            target = None
            if m[1].startswith(("s_branch", "s_cbranch")):
                t = re.search(r"<.*?(?:\+0x([0-9a-f]+))?>", m[4])
                target = base + int(t[1] or "0", 16)
            cur.append((int(m[3], 16), m[1], m[2], target))
    return funcs


def _touched_in_flight(ins, heed_waits=True):
    """Instructions that name a register which an LDS read may still have to write; LDS reads come back in order."""
    at = {a: i for i, (a, *_) in enumerate(ins)}
    succ = []
    for i, (_, op, _, target) in enumerate(ins):
        nxt = [] if op in ("s_endpgm", "s_branch") else [i + 1]
        succ.append([j for j in nxt + ([at[target]] if target is not None else []) if j < len(ins)])
    joins = {j for i, s in enumerate(succ) for j in s if s != [i + 1]} | {i + 1 for i, s in enumerate(succ) if s != [i + 1]}
    state, work, found = {0: {}}, [0], set()       # register -> LDS and scalar memory operations issued behind its read
    while work:
        i = work.pop()
        st = dict(state[i])
        while True:
            _, op, args, _ = ins[i]
            if not op.startswith("s_") and any(r in st for r in _regs(args)):
                found.add((op, args))
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                left = int(m[1]) if m else (0 if "cnt" not in args else None)
                if left is not None and heed_waits:
                    st = {r: n for r, n in st.items() if n < left}
            elif op.startswith(("ds_", "s_load", "s_buffer_load")):
                st = {r: min(n + 1, 15) for r, n in st.items()}
                if op.startswith("ds_read"):
                    st.update((r, 0) for r in _regs(args.split(",")[0]))
            if succ[i] == [i + 1] and i + 1 not in joins:
                i += 1
                continue
            for j in succ[i]:
                old = state.get(j)
                if old is None or any(old.get(r, 99) > n for r, n in st.items()):
                    state[j] = {r: min(st.get(r, 99), (old or {}).get(r, 99)) for r in st.keys() | (old or {}).keys()}
                    work.append(j)
            break
    return found


def test_no_register_is_used_while_a_read_into_it_is_under_way(code_objects):
    seen = 0
    for f in code_objects:
        for name, ins in _functions(f).items():
            if any(op.startswith("ds_read") for _, op, *_ in ins):
                seen += 1
                assert not (bad := _touched_in_flight(ins)), f"{name}: {sorted(bad)[:3]}"
                assert _touched_in_flight(ins, heed_waits=False), name      # the check itself: without the waits it does object
    assert seen > 80


def test_matrix_instructions_follow_vector_writes_of_their_operands_at_a_distance(code_objects):
    """Two wait states between a vector instruction and a matrix instruction that reads its result (what the compiler itself keeps)."""
    seen = 0
    for f in code_objects:
        for name, ins in _functions(f).items():
            for i, (_, op, args, _) in enumerate(ins):
                if not op.startswith("v_mfma"):
                    continue
                seen += 1
                read, states, j = _regs(",".join(args.split(",")[1:])), 0, i - 1
                while j >= 0 and states < 2:
                    _, o, a, _ = ins[j]
                    if o == "s_nop":
                        states += int(a, 0)
                    elif o.startswith("v_") and not o.startswith(("v_mfma", "v_cmp")):
                        wrote = _regs(a if o.startswith(("v_permlane", "v_swap")) else a.split(",")[0])
                        assert not wrote & read, f"{name}: {o} {a} in front of {op} {args}"
                    states += 1
                    j -= 1
    assert seen > 5000


def _loads_in_flight(ins):
    """{index of a barrier: most direct loads to LDS that may still be under way there}, over all paths to it.  Memory operations end in the
    order they were issued, so a load is done where a wait allows no more operations than were issued since; on the path with the fewest."""
    at = {a: i for i, (a, *_) in enumerate(ins)}
    succ = [[j for j in ([] if op in ("s_endpgm", "s_branch") else [i + 1]) + ([at[t]] if t is not None else []) if j < len(ins)]
            for i, (_, op, _, t) in enumerate(ins)]
    joins = {j for i, s in enumerate(succ) for j in s if s != [i + 1]} | {i + 1 for i, s in enumerate(succ) if s != [i + 1]}
    state, work, found, most = {0: ()}, [0], {}, 48       # operations issued since each direct load, the latest load first; 48 and more are let go
    while work:
        i = work.pop()
        st = list(state[i])
        while True:
            _, op, args, _ = ins[i]
            if op.startswith(("global_", "buffer_", "flat_")):
                st = ([0] if "lds" in op else []) + [n + 1 for n in st if n + 1 < most]
            elif op == "s_waitcnt" and "vmcnt" in args:
                left = int(re.search(r"vmcnt\((\d+)\)", args)[1])
                assert left <= most
                st = [n for n in st if n < left]
            elif op == "s_barrier":
                found[i] = max(found.get(i, 0), len(st))
            if succ[i] == [i + 1] and i + 1 not in joins:
                i += 1
                continue
            for j in succ[i]:
                old = state.get(j)
                new = tuple(st) if old is None else tuple(min(p) for p in zip(st, old)) + (tuple(st) if len(st) > len(old) else old)[min(len(st), len(old)):]
                if new != old:
                    state[j] = new
                    work.append(j)
            break
    return found


def test_waits_of_the_resident_workgroups_cover_the_next_slab(code_objects):
    """The kernel of resident workgroups names, in front of each barrier, how many memory operations may still be under way: at most the
    loads of the slabs behind the next one.  The stores and side inputs it counts beside them must have been issued since on every path."""
    seen = 0
    for f in code_objects:
        for name, ins in _functions(f).items():
            m = re.search(r"gemm_bf16_flow_kernelILi(\d+)ELi(\d+)ELi(\d+)E", name)
            if not m:
                continue
            bm, bn, bufs = map(int, m.groups())
            behind = (bufs - 2) * (bm + bn) * 128 // 4096
            found = _loads_in_flight(ins)
            assert max(found.values()) <= behind, (name, sorted(found.values())[-3:])
            # the check itself: without the waits there are more
            assert max(_loads_in_flight([(a, "s_nop" if op == "s_waitcnt" else op, args, t) for a, op, args, t in ins]).values()) > behind
            seen += len(found)
    assert seen > 100
