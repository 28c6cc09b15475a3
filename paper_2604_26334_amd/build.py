"""Build libpshard.so (host planner/scheduler/packer + HIP kernels and executor) for gfx950.

Besides compiling, the build CHECKS what the hand-placed waits of the MFMA GEMM rely on, from the
compiler's own output for kernels.hip, and fails if it does not hold:
  - the kernels that must not be placed beside a gather copy use LDS (NEEDS_LDS);
  - no kernel of the matmul / attention families uses scratch memory or spills a register (a spill
    reload is a vector-memory operation and would be counted by `s_waitcnt vmcnt(n)` like a prefetch);
  - in every gemm_w4_kernel, a vmcnt(0) stands between the opening prefetches and the first barrier; every later stretch
    between two barriers that ends in a counted wait vmcnt(n > 0) issues exactly the loads of one
    prefetch, LDS fills first, and n is the count the kernel's ring depth implies; nothing else
    touches vector memory inside the ring (a grouped kernel holds the rings of up to three tiles: each is there, told by its opening
    prefetches, and its steps are checked against its own counts);
  - in every gemm_w4_kernel of two K parts, on every path to a write into LDS (the exchange of the parts' sums, which
    lies over the ring's stages), a vmcnt(0) and then a barrier stand behind the last LDS fill: no wave's fill can
    land on another wave's sums;
  - in every gemm_kslice_kernel, on every path: a wave reads a ring slot only once the slot's fill has landed, refills it only
    once those reads have returned, and meets the first barrier with every fill landed and read.
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.environ.get("PS_LIB_OUT", os.path.join(HERE, "libpshard.so"))
BUILD = os.path.join(HERE, "_build")
SOURCES = ["planner.cpp", "schedule.cpp", "pack.cpp", "cpu_backend.cpp", "profile_db.cpp", "kernels.hip", "stack.hip", "profile.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -ffp-contract=off: results must not depend on which kernel a device function was inlined into
# (the one-token kernel variants have to agree bit for bit on every placement); fused multiply-adds
# are written out with fmaf where they are wanted
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC] + os.environ.get("PS_EXTRA_FLAGS", "").split()
CHECKED = "kernels.hip"      # the source whose kernels are checked
# kept off the CUs a gather copy holds (the GEMM, the few-token GEMV and the chunk attention by LDS given at launch, which
# the remarks do not show)
NEEDS_LDS = ("gemv_w4_kernel", "attn_decode_kernel", "splitk_epilogue_resid_rinv_kernel",
             "splitk_epilogue_resid_quarters_kernel", "splitk_epilogue_norm_kernel")
NO_SCRATCH = ("gemm_w4_kernel", "gemm_w4_upload_kernel", "gemm_kslice_kernel", "gemv_w4_kernel", "gemv_mt_kernel", "attn_decode_kernel", "attn_combine_kernel", "attn_chunk_kernel", "attn_combine_chunk_kernel")


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), err[-4000:]))
    return r.stderr


def _compile(src):
    obj = os.path.join(BUILD, src + ".o")
    hip = ["-x", "hip"] if src.endswith(".hip") else []
    remarks = ["-Rpass-analysis=kernel-resource-usage"] if src == CHECKED else []
    err = _run([HIPCC] + FLAGS + hip + remarks + ["-c", os.path.join(CSRC, src), "-o", obj])
    if src == CHECKED:
        check_resource_usage(err)
    else:
        err = "\n".join(l for l in err.splitlines() if "packed-fp32-ops" not in l)
        if err.strip():
            sys.stderr.write(err + "\n")
    return obj


def _isa(src):
    """Device assembly of one HIP source (a second, device-only compile next to the object build)."""
    out = os.path.join(BUILD, src + ".s")
    _run([HIPCC] + FLAGS + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out])
    return out


def check_resource_usage(remarks):
    """The compiler's per-kernel resource remarks: matmul and attention kernels use no scratch, and the
    gather copy kernel holds a CU's whole LDS (what keeps matmul workgroups off the CUs it reads PCIe from: they need some)."""
    name, bad, seen, gather_lds = None, [], 0, None
    for ln in remarks.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", ln)
        if m:
            name = m.group(1)
            seen += any(k in name for k in NO_SCRATCH)
            continue
        m = re.search(r"remark:\s+LDS Size \[bytes/block\]: (\d+)", ln)
        if m and name and "h2d_gather_kernel" in name:
            gather_lds = int(m.group(1))
        if m and name and any(k in name for k in NEEDS_LDS) and int(m.group(1)) == 0:
            bad.append("%s: no LDS, so it could be placed beside a gather copy" % name)
        m = re.search(r"remark:\s+(ScratchSize \[bytes/lane\]|SGPRs Spill|VGPRs Spill): (\d+)", ln)
        if m and name and any(k in name for k in NO_SCRATCH) and int(m.group(2)) != 0:
            bad.append("%s: %s = %s" % (name, m.group(1), m.group(2)))
    if seen == 0:
        raise RuntimeError("build check: no resource-usage remarks for the matmul kernels (compiler flag ignored?)")
    if bad:
        raise RuntimeError("build check: scratch / spills in kernels that must have none, or no LDS in one that must have some:\n  " + "\n  ".join(bad))
    if gather_lds != 160 * 1024:
        raise RuntimeError("build check: h2d_gather_kernel allocates %s B of LDS, not the CU's 163840" % gather_lds)


def gemm_wait_counts(mt, nw, at=2, ks=1):
    """(loads per prefetch, LDS fills among them, counted wait of a steady step) of gemm_w4_kernel<.., at, mt, .., nw, ks>."""
    nwr = nw // ks
    nfill = mt // (4 * nwr)
    lpi = nfill + at
    depth = (3 if mt <= 128 else 2 if mt <= 160 else 1) if nwr == 8 else (2 if mt <= 64 else 1)
    early = depth >= 3
    land = depth - 2 if early else depth - 1
    return lpi, nfill, land * lpi + (at if early else 0)


def blocks_of(body):
    """(labels in order, instructions of each) of a kernel's text."""
    blocks, order, cur = {"": []}, [""], ""
    for ln in body.splitlines():
        ln = ln.split(";")[0].strip()
        m = re.match(r"(\.LBB\w+):", ln)
        if m:
            cur = m.group(1)
            blocks[cur] = []
            order.append(cur)
        elif ln and not ln.startswith("."):
            blocks[cur].append(ln)
    return order, blocks


def lds_writes_behind_fills(body):
    """LDS writes of a kernel's text that some path reaches while a fill (a load straight into LDS) may still be in flight
    in this or another wave.  Per path: a fill leaves 2, vmcnt(0) turns 2 into 1 (this wave's have landed), a barrier
    turns 1 into 0 (everyone's have: all waves run the same steps).  A counted wait changes nothing."""
    order, blocks = blocks_of(body)
    bad, seen, todo = [], {}, [("", 0)]
    while todo:
        name, state = todo.pop()
        if seen.get(name, -1) >= state:
            continue
        seen[name] = state
        falls = True
        for ln in blocks[name]:
            ins = ln.split()[0]
            if ins.startswith("buffer_load") and re.search(r"\blds\b", ln):
                state = 2
            elif ins == "s_waitcnt" and re.search(r"vmcnt\(0\)", ln):
                state = min(state, 1)
            elif ins == "s_barrier":
                state = 0 if state == 1 else state
            elif ins.startswith("ds_write") and state:
                bad.append(ln)
            elif ins.startswith("s_cbranch"):
                todo.append((ln.split()[-1], state))
            elif ins == "s_branch":
                todo.append((ln.split()[-1], state))
                falls = False
                break
            elif ins == "s_endpgm":
                falls = False
                break
        if falls and order.index(name) + 1 < len(order):
            todo.append((order[order.index(name) + 1], state))
    return sorted(set(bad))


def kslice_ring_faults(body, nmt):
    """The first thing that some path of gemm_kslice_kernel's text up to its first barrier does against the ring of `nmt` slots
    that each wave keeps (none: empty): four fills to a slot and four reads from it, slot after slot; a read before the slot's fill has landed (loads return in the
    order of their issue, vmcnt counts those still out), a fill before the reads of what was there have returned, a fill that
    is out or unread at the barrier.  Where a path goes round the loop, only where the ring stands and what is out counts."""
    order, blocks = blocks_of(body)
    cap, seen = 4 * nmt, set()
    todo = [("", (), 0, 0, False)]    # label, loads out (slot or -1 each), fills issued (mod the ring), fills not read yet, reads out
    while todo:
        at = todo.pop()
        if at in seen:
            continue
        seen.add(at)
        if len(seen) > 10000:
            return ["more paths than such a walk has"]
        name, out, nf, unread, reads = at
        ended = False
        for ln in blocks[name]:
            ins = ln.split()[0]
            if ins.startswith("buffer_load") and re.search(r"\blds\b", ln):
                if reads:
                    return ["a fill while reads are out"]
                if unread >= cap:
                    return ["a fill of a slot that was not read"]
                out, nf, unread = out + (nf // 4,), (nf + 1) % cap, unread + 1
            elif re.match(r"(buffer_|global_|flat_|scratch_)", ins):
                out += (-1,)
            elif ins == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", ln)
                if m:
                    out = out[max(0, len(out) - int(m.group(1))):]
                if "lgkmcnt(0)" in ln:
                    reads = False
            elif ins.startswith("ds_"):
                if ins != "ds_read_b128" or unread <= 0:
                    return [ins + " where an operand of a filled slot is read"]
                elif (nf - unread) % cap // 4 in out:
                    return ["a read of a slot whose fill may be out"]
                unread, reads = unread - 1, True
            elif ins == "s_barrier":
                if unread or any(x >= 0 for x in out):
                    return ["a barrier with fills out or unread"]
                ended = True
                break
            elif ins.startswith("s_cbranch"):
                todo.append((ln.split()[-1], out, nf, unread, reads))
            elif ins == "s_branch":
                todo.append((ln.split()[-1], out, nf, unread, reads))
                ended = True
                break
            elif ins == "s_endpgm":
                return ["an end before the slices meet"]
            if len(out) > 64:
                return ["more loads out than vmcnt counts"]
        if not ended:
            if order.index(name) + 1 == len(order):
                return ["no barrier"]
            todo.append((order[order.index(name) + 1], out, nf, unread, reads))
    return []


def check_kslice_isa(path):
    """The invariant behind gemm_kslice_kernel's hand-counted waits, read off the generated code."""
    txt = open(path).read()
    funcs = re.findall(r"^(_ZN2ps18gemm_kslice_kernelILi\d+ELi(\d+)E\w+):[^\n]*\n(.*?)\n\.Lfunc_end", txt, flags=re.S | re.M)
    if not funcs:
        raise RuntimeError("build check: no gemm_kslice_kernel in " + path)
    bad = [(mangled, kslice_ring_faults(body, int(nmt))) for mangled, nmt, body in funcs]
    if any(faults for _, faults in bad):
        raise RuntimeError("build check: rings of K slices:\n  " + "\n  ".join("%s: %s" % (m, ", ".join(f)) for m, f in bad if f))
    return len(funcs)


def check_gemm_isa(path):
    """The invariant behind the GEMM's hand-counted waits, read off the generated code."""
    txt = open(path).read()
    funcs = re.findall(r"^(_ZN2ps(?:14gemm_w4_kernel|21gemm_w4_upload_kernel)\w+):[^\n]*\n(.*?)\n\.Lfunc_end", txt, flags=re.S | re.M)
    if not funcs:
        raise RuntimeError("build check: no gemm_w4_kernel in " + path)
    bad = []
    for mangled, body in funcs:
        m = re.match(r"_ZN2ps14gemm_w4_kernelILi\d+ELi(\d+)ELi(\d+)ELb([01])ELi(\d+)(?:ELi(\d+))?(?:ELb[01])?EEE", mangled)
        up = re.match(r"_ZN2ps21gemm_w4_upload_kernelILi(\d+)EEE", mangled)
        if not m and not up:
            bad.append(mangled + ": unexpected template arguments")
            continue
        at, mt, nw, ks = (int(m.group(k) or 1) for k in (1, 2, 4, 5)) if m else (2, int(up.group(1)), 4, 1)
        # an expert's workgroups may take one of the two tiles below the launch's: three rings in one kernel
        less = {32: 16, 48: 32, 64: 48, 96: 64, 128: 96} if m and m.group(3) == "1" else {}
        tiles = [t for t in (mt, less.get(mt), less.get(less.get(mt))) if t]
        counts = {t: gemm_wait_counts(t, nw, at, ks) for t in tiles}
        # by its opening prefetches: two with the first's scales (the rings of four waves with counted waits)
        openings = {2 * counts[t][1] + at: t for t in tiles if len(tiles) > 1 and counts[t][2]}
        tile, found = (None if len(tiles) > 1 else mt), set()
        segs, cur = [], []
        for ln in body.splitlines():
            f = ln.split()
            if not f:
                continue
            ins = f[0]
            if ins == "s_barrier":
                segs.append(cur)
                cur = []
            elif re.match(r"(buffer_|global_|flat_|scratch_)", ins):
                cur.append("lds" if (ins.startswith("buffer_load") and re.search(r"\blds\b", ln)) else ins)
            elif ins == "s_waitcnt" and "vmcnt" in ln:
                cur.append(int(re.search(r"vmcnt\((\d+)\)", ln).group(1)))
        segs.append(cur)        # the epilogue, after the last barrier
        if any(isinstance(x, str) and (x.startswith("scratch_") or x.startswith("flat_")) for s in segs for x in s):
            bad.append(mangled + ": scratch or flat memory instruction")
        if len(segs) < 3:
            bad.append(mangled + ": no barrier-delimited ring found")
            continue
        # (waits the compiler adds behind it for its own bookkeeping change nothing)
        last_load = max([k for k, x in enumerate(segs[0]) if isinstance(x, str)], default=-1)
        if 0 not in segs[0][last_load + 1:]:
            bad.append(mangled + ": no vmcnt(0) between the opening prefetches and the first barrier")
        steps = 0
        for k, s in enumerate(segs[:-1]):
            loads = [x for x in s if isinstance(x, str)]
            waits = [x for x in s if isinstance(x, int)]
            if "lds" not in loads:
                continue       # not a ring step
            opening = loads[loads.index("lds"):]
            if len(tiles) > 1 and waits and waits[-1] == 0 and len(opening) - opening.count("lds") == 2 * at:
                tile = openings.get(opening.count("lds"))
                if tile in found or tile is None:
                    bad.append("%s: opening prefetches of %s" % (mangled, opening))
                found.add(tile)
            if k == 0:
                continue
            steps += 1
            if not waits:
                bad.append(mangled + ": ring step without a vmcnt wait")
            elif waits[-1] == 0:       # the opening prefetches of a further tile
                if 0 not in s[max(k for k, x in enumerate(s) if isinstance(x, str) and x == "lds") + 1:]:
                    bad.append(mangled + ": LDS fills that no vmcnt(0) and no counted wait stands behind")
            else:
                # every prefetch: the activation fills, then one code load per tile; one prefetch in eight
                # starts with a scale fill per tile (a branch: the text holds it either way)
                nl = loads.count("lds")
                lpi, nfill, in_flight = counts.get(tile, (0, 0, 0))
                if waits[-1] != in_flight or nl not in (nfill, nfill + at) or loads[:nl] != ["lds"] * nl or len(loads) != nl + at:
                    bad.append("%s: a counted ring step of the %s-token ring issues %s and waits for vmcnt(%d), expected %d (+ %d) LDS fills, %d weight loads and vmcnt(%d)" % (
                        mangled, tile, loads, waits[-1], nfill, at, at, in_flight))
                if any(not x.startswith("buffer_load") for x in loads if x != "lds"):
                    bad.append(mangled + ": a ring step touches vector memory with something other than its prefetch")
        if steps == 0:
            bad.append(mangled + ": no ring step recognised")
        missing = [t for t in tiles if counts[t][2] and t not in found] if len(tiles) > 1 else []
        if missing:
            bad.append("%s: no counted ring step of the tiles %s" % (mangled, missing))
        if ks == 2:
            over = lds_writes_behind_fills(body)
            if over:
                bad.append("%s: %d writes into LDS with a fill of the ring possibly in flight, e.g. %s" % (mangled, len(over), over[0]))
    if bad:
        raise RuntimeError("build check: the GEMM's counted waits do not match the generated code:\n  " + "\n  ".join(bad))
    return len(funcs)


def build():
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=6) as ex:
        isa = ex.submit(_isa, CHECKED)
        objs = list(ex.map(_compile, SOURCES))
        n = check_gemm_isa(isa.result()) + check_kslice_isa(isa.result())
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    sys.stderr.write("build checks passed: no scratch in the matmul/attention kernels; %d GEMM instantiations match their wait counts\n" % n)
    return LIB


if __name__ == "__main__":
    print(build())
