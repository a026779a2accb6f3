"""In-tree builds: the HIP C-ABI library (hipcc, gfx950) and the input-generator library (gcc)."""
import os
import subprocess

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
REPO_DIR = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIBFGATTN = os.path.join(PKG_DIR, "libfgattn.so")
LIBFGW = os.path.join(PKG_DIR, "workloads", "libfgw.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HIP_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-fno-honor-nans",
]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("build failed: %s\n%s" % (" ".join(cmd), r.stdout))
    return r.stdout


def build_workloads(force=True):
    src = os.path.join(PKG_DIR, "workloads", "fgw_gen.c")
    if force or not os.path.exists(LIBFGW):
        _run(["gcc", "-O2", "-std=c11", "-fopenmp", "-fPIC", "-shared", src, "-o", LIBFGW, "-lm"])
    return LIBFGW


def check_m0_writes(asm_path):
    """The gathers of the forward kernel set the LDS-DMA base register M0 in one inline-assembly statement and rely
    on it in the following ones; nothing the compiler emits in between may write M0.  Every mention of M0 in the
    device assembly must therefore be one of the kernel's own marked `s_mov_b32 m0` lines."""
    import re
    tok = re.compile(r"\bm0\b")
    with open(asm_path) as f:
        for n, line in enumerate(f, 1):
            code = line.split(";", 1)[0]
            if tok.search(code) and "fg_m0" not in line:
                raise RuntimeError("%s:%d: M0 is touched outside the kernel's own gather statements: %s" %
                                   (asm_path, n, line.strip()))


def check_inline_asm_hazards(asm_path):
    """Vector-memory instructions written as inline assembly (the LDS-DMA gathers, the untracked id loads) get none of
    the wait states the compiler inserts for hardware hazards.  The one that could apply to them: a vector-ALU
    instruction that writes a scalar register (v_readfirstlane, v_readlane, a compare with a scalar destination) must be
    five wait states ahead of a vector-memory instruction that reads that register as its base.  The kernels keep such
    bases in scalar registers from the start, so no such write should be anywhere near; this scan fails the build if
    one ever is."""
    import re
    sreg = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")
    window = []   # (wait states this instruction contributes, scalar registers a vector-ALU instruction writes)
    with open(asm_path) as f:
        for n, line in enumerate(f, 1):
            code = line.split(";", 1)[0].strip()
            if not code or code.startswith(".") or code.endswith(":"):
                continue
            op = code.split()[0]
            if op.startswith("global_load") or op.startswith("global_store"):
                m = sreg.search(code.split(None, 1)[1]) if " " in code else None
                if m:
                    lo, hi = (int(m.group(1)), int(m.group(2))) if m.group(1) else (int(m.group(3)), int(m.group(3)))
                    states = 0
                    for w, written in reversed(window):
                        if states >= 5:
                            break
                        if any(lo <= r <= hi for r in written):
                            raise RuntimeError("%s:%d: a vector-ALU write of s%s is only %d wait states ahead of %s" %
                                               (asm_path, n, sorted(written), states, code))
                        states += w
            written = set()
            if op.startswith("v_"):
                first = code.split(None, 1)[1].split(",")[0] if " " in code else ""
                m = sreg.fullmatch(first.strip())
                if m:
                    written = set(range(int(m.group(1)), int(m.group(2)) + 1)) if m.group(1) else {int(m.group(3))}
            states = 1
            if op == "s_nop":
                states = int(code.split()[1], 0) + 1
            window.append((states, written))
            if len(window) > 8:
                window.pop(0)


def check_untracked_loads(asm_path):
    """The compiler takes the target register of a load written as inline assembly (marked fg_id) as written at once, and
    as free when it is not read again; the load writes it later.  Every path from such a load must therefore come to an
    `s_waitcnt vmcnt(n)` that covers it (at most n vector-memory operations were issued after it; they complete in order)
    before anything reads or writes the register.  Follows all paths of every function: per instruction, the registers
    that may still be waiting and the fewest operations issued since.  Branches on a condition that was just set to a
    constant (the compiler joins loop exits that way) are followed in their one direction.  Returns how many marked loads
    it followed."""
    import re
    pair = re.compile(r"s\[(\d+):(\d+)\]")
    sregs = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")
    vreg = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")
    vmcnt = re.compile(r"vmcnt\((\d+)\)")
    vmem = ("global_", "buffer_", "flat_", "scratch_")

    def regs(text):
        found = set()
        for lo, hi, one in vreg.findall(text):
            found.update(range(int(lo), int(hi) + 1) if lo else (int(one),))
        return found

    def constants(known, op, args):
        """What is known of scalar pairs and vcc after an instruction: all ones / nothing set (kept: True / False)."""
        ops = [x.strip() for x in args.split(",")]
        if op == "s_mov_b64" and pair.fullmatch(ops[0]) and ops[1] in ("-1", "0"):
            known = {k: v for k, v in known.items() if not clash(k, ops[0])}
            known[ops[0]] = ops[1] == "-1"
        elif op in ("s_and_b64", "s_andn2_b64") and ops[:2] == ["vcc", "exec"]:
            known = {k: v for k, v in known.items() if k != "vcc"}
            if ops[2] in known:
                known["vcc"] = known[ops[2]] == (op == "s_and_b64")
        elif not op.startswith("s_cbranch") and not op.startswith("v_cndmask"):
            known = {k: v for k, v in known.items() if not clash(k, args)}
        return known

    def clash(key, args):
        if key == "vcc":
            return "vcc" in args
        lo, hi = map(int, pair.fullmatch(key).groups())
        return any(int(a or c) <= hi and int(b or c) >= lo for a, b, c in sregs.findall(args))

    def follow(code, labels):
        """code: (line number, opcode, operands, marked)"""
        # (instruction, what is known of scalar conditions) -> {register: fewest vector-memory operations since its load}
        waiting = {(0, frozenset()): {}}
        todo = list(waiting)
        while todo:
            at, known = place = todo.pop()
            n, op, args, marked = code[at]
            state, known = dict(waiting[place]), constants(dict(known), op, args)
            touched = regs(args) & state.keys()
            if touched:
                raise RuntimeError("%s:%d: v%s is touched while a load into it may be in flight: %s %s" %
                                   (asm_path, n, sorted(touched), op, args))
            if op == "s_waitcnt":
                m = vmcnt.search(args)
                limit = int(m.group(1)) if m else (0 if args.strip() == "0" else 64)
                state = {r: c for r, c in state.items() if c < limit}
            elif op.startswith(vmem):
                state = {r: min(c + 1, 63) for r, c in state.items()}
                if marked:
                    (target,) = regs(args.split(",")[0])
                    state[target] = 0
            after = []
            if op.startswith(("s_branch", "s_cbranch")):
                after.append(labels[args.strip()])
            elif op.startswith(("s_setpc", "s_swappc", "s_call")):
                raise RuntimeError("%s:%d: %s is not followed" % (asm_path, n, op))
            # (a forward s_cbranch_execnz ends a block that some lanes run, or it would have been skipped: always taken)
            always = op in ("s_branch", "s_endpgm") or (op == "s_cbranch_execnz" and after[0] > at)
            if op in ("s_cbranch_vccnz", "s_cbranch_vccz") and "vcc" in known:
                always = known["vcc"] == (op == "s_cbranch_vccnz")
                if not always:
                    after = []
            if not always and at + 1 < len(code):
                after.append(at + 1)
            for b in [(b, frozenset(known.items())) for b in after]:
                old = waiting.get(b)
                new = state if old is None else {r: min(old.get(r, 64), state.get(r, 64)) for r in old.keys() | state.keys()}
                if new != old:
                    waiting[b] = new
                    todo.append(b)

    loads, code, labels = 0, [], {}
    with open(asm_path) as f:
        for n, line in enumerate(f, 1):
            text, _, comment = line.partition(";")
            text = text.strip()
            if text.startswith(".Lfunc_end"):
                if any(marked for _, _, _, marked in code):
                    follow(code, labels)
                code, labels = [], {}
            elif text.endswith(":"):
                labels[text[:-1]] = len(code)
            elif text and not text.startswith("."):
                op, _, args = text.partition(" ") if " " in text else text.partition("\t")
                marked = "fg_id" in comment and op.startswith("global_load")
                loads += marked
                code.append((n, op, args, marked))
    return loads


def check_spills(asm_path):
    """A forward kernel that spills vector registers reloads them through the counter its gathers are waited for with.
    One register is tolerated (it is reloaded once per item where the key loop has no room)."""
    import re
    name = None
    with open(asm_path) as f:
        for line in f:
            m = re.match(r"\s+\.(name|vgpr_spill_count):\s+(\S+)", line)
            if m and m.group(1) == "name":
                name = m.group(2)
            elif m and "fgattn_fwd_kernel" in (name or "") and int(m.group(2)) > 1:
                raise RuntimeError("%s: %s spills %s vector registers" % (asm_path, name, m.group(2)))


def check_rounding_mode(asm_path):
    """The histogram of the mask selection forms its weights by 64-bit float instructions written as inline assembly, under a
    rounding mode that the kernel sets once at its start and that the compiler does not know of.  A 64-bit float
    instruction of the compiler's own in such a kernel would be rounded wrongly, or the compiler would set the mode back ahead of it;
    and the statement in a kernel that does not set the mode would round to nearest.  Per function: one write of the mode at
    most, ahead of every 64-bit float instruction; with it, all of these are inline assembly, without it, none is.  Returns how many
    functions set the mode."""
    import re
    double = re.compile(r"v_\w*f64")
    found, mode, inline, first = 0, None, False, None
    with open(asm_path) as f:
        for n, line in enumerate(f, 1):
            if "#ASMSTART" in line or "#ASMEND" in line:
                inline = "#ASMSTART" in line
                continue
            text = line.split(";", 1)[0].strip()
            op = text.split()[0] if text else ""
            if text.startswith(".Lfunc_end"):
                found += mode is not None
                mode, first = None, None
            elif op.startswith(("s_setreg", "s_round_mode", "s_denorm_mode")):
                if mode is not None or first is not None or "HW_REG_MODE, 2, 2), 3" not in text:
                    raise RuntimeError("%s:%d: the mode of float operations is written again, late or otherwise: %s" % (asm_path, n, text))
                mode = n
            elif double.match(op):
                first = n if first is None else first
                if inline != (mode is not None):
                    raise RuntimeError("%s:%d: a 64-bit float instruction under the wrong rounding mode: %s" % (asm_path, n, text))
    return found


def build_hip(force=True, extra_flags=()):
    """Compile every .hip translation unit for gfx950 (in parallel) and link libfgattn.so in-tree."""
    from concurrent.futures import ThreadPoolExecutor
    srcs = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]
    if not force and os.path.exists(LIBFGATTN):
        return LIBFGATTN
    objdir = os.path.join(PKG_DIR, "_build")
    os.makedirs(objdir, exist_ok=True)
    common = [f for f in HIP_FLAGS if f != "-shared"] + list(extra_flags) + \
        ["-save-temps=obj", "-I", os.path.join(REPO_DIR, "include"), "-I", CSRC]
    objs = [os.path.join(objdir, os.path.basename(s)[:-4] + ".o") for s in srcs]
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        list(ex.map(lambda so: _run([HIPCC] + common + ["-c", so[0], "-o", so[1]]), zip(srcs, objs)))
    for f in sorted(os.listdir(objdir)):
        if f.endswith("-gfx950.s"):
            check_m0_writes(os.path.join(objdir, f))
            check_inline_asm_hazards(os.path.join(objdir, f))
            check_untracked_loads(os.path.join(objdir, f))
            check_spills(os.path.join(objdir, f))
            check_rounding_mode(os.path.join(objdir, f))
        elif not f.endswith(".o"):
            os.remove(os.path.join(objdir, f))   # other intermediates of -save-temps
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIBFGATTN])
    return LIBFGATTN


def source_id():
    """What a measurement script prints so that its table can be tied to a tree: the git commit if this is a
    checkout (with '+' if tracked files differ from it), and a digest of the kernel and generator sources, which can
    be recomputed from any copy of the files."""
    import hashlib
    head = "unknown"
    try:
        r = subprocess.run(["git", "-C", REPO_DIR, "rev-parse", "--short=12", "HEAD"], stdout=subprocess.PIPE,
                           stderr=subprocess.DEVNULL, text=True)
        if r.returncode == 0 and r.stdout.strip():
            head = r.stdout.strip()
            d = subprocess.run(["git", "-C", REPO_DIR, "status", "--porcelain", "--untracked-files=no"],
                               stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True)
            if d.returncode == 0 and d.stdout.strip():
                head += "+"
    except OSError:
        pass
    h = hashlib.sha256()
    files = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith((".hip", ".hpp"))]
    files += [os.path.join(REPO_DIR, "include", "fgattn.h"), os.path.join(PKG_DIR, "workloads", "fgw_gen.c")]
    for path in files:
        with open(path, "rb") as f:
            h.update(os.path.basename(path).encode() + b"\0" + f.read())
    return {"git_head": head, "source_sha256": h.hexdigest()[:16]}
