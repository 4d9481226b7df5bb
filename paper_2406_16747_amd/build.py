"""Builds libsparsek.so (HIP, gfx950) in-tree with hipcc.  No GPU is needed to build.

Besides the library the build writes libsparsek.toolchain.json: the compiler it used and the result of a check of
the generated code.  Three kernels (attention forward, mask backward, dK/dV) issue direct-to-LDS loads from inline
assembly that sets the M0 register itself; that is only sound while the compiler keeps no value of its own in M0
inside those kernels.  The check reads the device assembly of every translation unit and accepts a mention of M0
only in the three-instruction pattern of those loads.  A second check looks for barriers that an LDS write can reach
without a wait: the compiler has left such waits out at the head of loops.  A third one looks at matrix products written
as inline assembly (dK/dV): the compiler does not know that they are products and keeps none of their distances.
"""
import json
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsparsek.so")
OBJ = os.path.join(HERE, "_build")
SIDECAR = os.path.join(HERE, "libsparsek.toolchain.json")

# The compiler the kernels' hand-written M0 handling was validated with (GPU parity tests green).  Another version
# is not wrong by itself -- check_m0 below looks at the code it generates -- but the tests ask for a fresh validation.
VALIDATED_HIPCC = "HIP version: 7.2.26015"

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-result",
    # packed-fp32 VALU forms are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def check_m0(asm_path):
    """Per kernel of a device assembly file: the mentions of M0 are either all inside inline-assembly regions (the
    hand-written direct-to-LDS loads of attn_tiles.hpp, which set M0 themselves) or all outside (M0 managed by the
    compiler, e.g. for the builtin form of the same loads).  A kernel with both would let the hand-written loads
    clobber a value the compiler keeps in M0.  Returns {kernel: number of hand-written loads}; raises on a mix."""
    found = {}
    name, in_asm, ours, theirs = None, False, 0, []
    for raw in open(asm_path, errors="replace"):
        ln = raw.strip()
        if ln.startswith(";;#ASMSTART"):
            in_asm = True
        elif ln.startswith(";;#ASMEND"):
            in_asm = False
        elif ln.startswith(".Lfunc_end"):
            if ours and theirs:
                raise RuntimeError("%s: kernel %s sets M0 by hand (%d loads) while the compiler uses it too: `%s`"
                                   % (os.path.basename(asm_path), name, ours, theirs[0]))
            if ours:
                found[name] = ours
            name, ours, theirs = None, 0, []
        elif re.match(r"^[A-Za-z_][\w$.]*:", ln) and not ln.startswith(".L"):
            name = ln.split(":")[0]
        else:
            code = ln.split(";")[0]
            if re.search(r"\bm0\b", code):
                if in_asm:
                    ours += 1 if code.startswith("s_mov_b32 m0") else 0
                else:
                    theirs.append(code)
    return found


def check_waits(asm_path):
    """Raises if an LDS write or atomic of some kernel can reach a barrier without a wait (s_waitcnt lgkmcnt(0)) on the
    way: another wave may then read what was there before.  Returns the number of barriers looked at."""
    count, name, code = 0, None, []
    for raw in open(asm_path, errors="replace"):
        ln = raw.split(";")[0].strip()
        if re.match(r"^[A-Za-z_][\w$.]*:$", ln) and not ln.startswith(".L"):
            name, code = ln[:-1], []
        elif raw.startswith(".Lfunc_end"):
            bad = _barriers_with_writes(code)
            if bad:
                raise RuntimeError("%s: an LDS write of kernel %s reaches a barrier without a wait (instruction %d)"
                                   % (os.path.basename(asm_path), name, bad[0]))
            count += code.count("s_barrier")
            code = []
        elif ln:
            code.append(ln)
    return count


def _barriers_with_writes(code):
    """Indexes of the barriers that an LDS write reaches without a wait, over all paths of a function's instructions."""
    label = {t[:-1]: i for i, t in enumerate(code) if t.endswith(":")}
    seen = [None] * len(code)   # whether a write may be under way ahead of the instruction
    work, bad = [(0, False)], set()
    while work:
        i, pending = work.pop()
        while i < len(code) and (seen[i] is None or (pending and not seen[i])):
            seen[i] = pending
            op, _, args = code[i].partition(" ")
            if op.startswith("ds_") and not re.match(r"ds_(read|bpermute|permute|swizzle)", op):
                pending = True
            elif op == "s_waitcnt" and "lgkmcnt(0)" in args or op == "s_swappc_b64":   # (a function starts with a wait)
                pending = False
            elif op == "s_barrier" and pending:
                bad.add(i)
            if re.match(r"s_c?branch", op) and args.strip() in label:
                work.append((label[args.strip()], pending))
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            i += 1
    return sorted(bad)


# Matrix products written by hand: states (instructions, s_nop counting for more) that have to lie between a product of 8
# passes and anything else that names its result, between a vector instruction and a product that reads what it wrote, and
# between one that writes EXEC and a product.
RESULT_STATES, OPERAND_STATES, EXEC_STATES = 12, 2, 4


def check_products(asm_path):
    """Raises if the code around a matrix product written as inline assembly does not keep the distances above, on some
    path.  Returns {kernel: number of such products}."""
    found, name, code, in_asm = {}, None, [], False
    for raw in open(asm_path, errors="replace"):
        ln = raw.strip()
        if ln.startswith(";;#ASMSTART"):
            in_asm = True
        elif ln.startswith(";;#ASMEND"):
            in_asm = False
        elif ln.startswith(".Lfunc_end"):
            count = sum(1 for ours, text in code if ours and text.startswith("v_mfma"))
            if count:
                bad = _products_at_fault(code)
                if bad:
                    raise RuntimeError("%s: kernel %s: %s" % (os.path.basename(asm_path), name, bad[0]))
                found[name] = count
            name, code = None, []
        elif re.match(r"^[A-Za-z_][\w$.]*:", ln) and not ln.startswith(".L"):
            name, code = ln.split(":")[0], []
        else:
            text = ln.split(";")[0].strip()
            if text and (text.endswith(":") or not text.startswith(".")):
                code.append((in_asm, text))
    return found


def _registers(operand):
    """The vector registers (v and a) an operand of an instruction names."""
    regs = set()
    for bank, one, first, last in re.findall(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", operand):
        regs |= {(bank, i) for i in (range(int(first), int(last) + 1) if first else (int(one),))}
    return regs


def _products_at_fault(code):
    """What breaks the distances, over all paths of a function's instructions, given as (inline assembly, text)."""
    steps, label = [], {}
    for i, (ours, text) in enumerate(code):
        op, _, args = text.partition(" ")
        operands = [_registers(x) for x in args.split(",")]
        named, read = set().union(*operands), set().union(*operands[1:])
        mfma, branch = op.startswith(("v_mfma", "v_smfma")), None
        if op.endswith(":"):
            label[op[:-1]] = i
        if re.match(r"s_c?branch", op):
            branch = args.strip()
        written = set()   # by a vector instruction that is no product
        if op.startswith("v_") and not mfma:
            written = named if "swap" in op else operands[0]
        states = 0 if op.endswith(":") else int(args, 0) + 1 if op == "s_nop" else 1
        # (a product that goes on with a sum names it as its first and its last operand, and nowhere else)
        tied = mfma and len(operands) >= 4 and operands[0] == operands[3] and not operands[0] & (operands[1] | operands[2])
        steps.append((ours, text, op, operands[0], named, read, mfma, tied, written, states, branch))
    # per instruction reached by a branch or at the start: what is under way, and for how many more states
    entry, work, faults = {0: {}}, [0], {}
    while work:
        i = work.pop()
        way = dict(entry[i])
        while i < len(steps):
            ours, text, op, first, named, read, mfma, tied, written, states, branch = steps[i]
            for (kind, what), left in way.items():
                if kind == "operand":
                    bad = ours and mfma and what in read
                elif kind == "exec":
                    bad = ours and mfma
                else:   # the result of a product: one of ours for everybody, another one for ours
                    bad = what & named and (kind == "our result" or (ours and mfma)) and not (mfma and tied and first == what)
                if bad:
                    faults[i] = "`%s` comes %d states too early after %s" % (
                        text, left, "a write of EXEC" if kind == "exec" else "a write of its operand" if kind == "operand"
                        else "a product into %s%d.." % min(what))
            if states:
                way = {key: left - states for key, left in way.items() if left > states}
            if mfma:
                way[("our result" if ours else "result", frozenset(first))] = RESULT_STATES
            for reg in written:
                way[("operand", reg)] = OPERAND_STATES
            if op.startswith("v_cmpx"):
                way[("exec", None)] = EXEC_STATES
            targets = [label[branch]] if branch in label else []
            if i + 1 < len(steps) and steps[i + 1][2].endswith(":") and op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                targets.append(i + 1)
            for t in targets:
                have = entry.get(t)
                merged = dict(have or {})
                for key, left in way.items():
                    merged[key] = max(left, merged.get(key, 0))
                if merged != have:
                    entry[t] = merged
                    work.append(t)
            if op in ("s_branch", "s_endpgm", "s_setpc_b64") or (targets and targets[-1] == i + 1):
                break
            i += 1
    return [faults[i] for i in sorted(faults)]


def build(verbose=False):
    """Compiles every .hip file and links the shared library.  Always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)

    def one(src):
        obj = os.path.join(OBJ, src[:-4] + ".o")
        cmd = [hipcc] + FLAGS + ["-save-temps=obj", "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, r.stderr[-4000:]))
        if verbose and r.stderr.strip():
            print(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(sources()))) as ex:
        objs = list(ex.map(one, sources()))
    tmp = LIB + ".tmp%d" % os.getpid()
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s" % r.stderr[-4000:])
    os.replace(tmp, LIB)
    version = subprocess.run([hipcc, "--version"], capture_output=True, text=True).stdout.strip()
    loads, products = {}, {}
    for src in sources():
        asm = os.path.join(OBJ, src[:-4] + "-hip-amdgcn-amd-amdhsa-gfx950.s")
        check_waits(asm)
        products.update(check_products(asm))
        n = check_m0(asm)
        if n:
            loads[src] = sum(n.values())
    with open(SIDECAR, "w") as f:
        json.dump({"hipcc_version": version.splitlines(), "flags": FLAGS,
                   "m0_check": "ok", "waits_check": "ok", "hand_written_products": sum(products.values()), "untracked_direct_to_lds_loads": loads}, f, indent=1)
    keep = {src[:-4] + ".o" for src in sources()}
    for name in os.listdir(OBJ):   # the intermediate files of -save-temps
        if name not in keep:
            os.remove(os.path.join(OBJ, name))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
