"""Static checks of the compiled gfx950 code.

scan(): a guard for scalar loads written as inline asm.  The compiler does not know that the
destination SGPRs of such a load are in flight until the next s_waitcnt lgkmcnt(0); the scan
walks every kernel linearly and reports any instruction that reads or writes an SGPR of an
inline-asm scalar load between its issue and that wait.  (Unconditional branches and s_endpgm
end a straight-line run.)  The kernels here fetch their wave-uniform operands with ordinary
constant-address-space loads, which the compiler tracks itself, so the scan finds no such load
at all; it stays in the build as a guard against one coming back.

asm_hazards(): wait states missing between an instruction of the compiler's and one written as asm.

kernel_stats(): spill counts and instruction histograms per kernel, for the code-generation
checks of the build.
"""
import re, sys

def regs(tok):
    tok = tok.strip()
    m = re.match(r'^s\[(\d+):(\d+)\]$', tok)
    if m: return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r'^s(\d+)$', tok)
    if m: return {int(m.group(1))}
    return set()

NO_SDST = ('s_cmp', 's_cbranch', 's_branch', 's_waitcnt', 's_barrier', 's_nop', 's_endpgm', 's_bitcmp',
           's_setprio', 's_sleep', 's_setreg', 's_sendmsg', 's_icache', 's_dcache', 's_store', 's_buffer_store')

def scan(path):
    """Returns a list of (kernel, line, text, 'reads'|'writes', registers, issue line)."""
    lines = open(path).read().split('\n')
    label_in = {}  # (kernel, label) -> loads in flight at some branch to that label
    for _ in range(4):  # a few sweeps so that states carried by backward branches settle
        out = set()
        kern, inflight, in_asm = None, [], False
        for i, l in enumerate(lines):
            t = l.strip()
            if t.startswith(';;#ASMSTART'): in_asm = True; continue
            if t.startswith(';;#ASMEND'): in_asm = False; continue
            m = re.match(r'^(_Z\w+):', t)
            if m: kern, inflight = m.group(1), []; continue
            m = re.match(r'^(\.LBB\w+):', t)
            if m:
                for e in label_in.get((kern, m.group(1)), []):
                    if e not in inflight: inflight.append(e)
                continue
            if not t or t[0] in ';.':
                continue
            t = t.split(';')[0].strip()
            op = t.split()[0]
            args = [a.strip() for a in t[len(op):].split(',')] if len(t) > len(op) else []
            if op == 's_waitcnt':
                if 'lgkmcnt(0)' in t: inflight = []
                continue
            if op.startswith(('s_cbranch', 's_branch')):
                tgt = label_in.setdefault((kern, args[0]), [])
                for e in inflight:
                    if e not in tgt: tgt.append(e)
                if op == 's_branch': inflight = []
                continue
            if op in ('s_endpgm', 's_setpc_b64'):
                inflight = []; continue
            dst = regs(args[0]) if args else set()
            writes = set()
            if op.startswith('s_') and not op.startswith(NO_SDST): writes = dst
            elif op.startswith(('v_readlane', 'v_readfirstlane')): writes = dst
            elif op.startswith('v_cmp') and op.endswith('_e64'): writes = dst
            srcs = set()
            for a in (args if not writes else args[1:]): srcs |= regs(a)
            for r, ln in inflight:
                if writes & set(r): out.add((kern, i + 1, t, 'writes', tuple(sorted(writes & set(r))), ln + 1))
                if srcs & set(r): out.add((kern, i + 1, t, 'reads', tuple(sorted(srcs & set(r))), ln + 1))
            if in_asm and op.startswith('s_load_dword'):
                inflight.append((tuple(sorted(dst)), i))
    return sorted(out, key=lambda e: e[1])

WAIT_SGPR_VALU, WAIT_SGPR_MEMORY, WAIT_LANES, WAIT_MFMA, WAIT_TRANS, WAIT_STORE = 2, 5, 2, 20, 1, 2
TRANS = ('v_rcp', 'v_rsq', 'v_sqrt', 'v_exp', 'v_log', 'v_sin', 'v_cos')

def operands(tok):
    """Registers of an operand, as 's4', 'v7', 'a3' or 'vcc'."""
    tok = tok.strip().lstrip('-').strip('|')
    if tok.startswith('vcc'): return {'vcc'}
    m = re.match(r'^([sva])\[(\d+):(\d+)\]$', tok)
    if m: return {m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    return {tok} if re.match(r'^[sva]\d+$', tok) else set()

def asm_hazards(path):
    """Wait states that the compiler leaves out because it does not look into an asm statement.

    The vector ALU does not interlock some of its results: a scalar register that it has written (a
    compare's mask, v_readlane) needs two wait states before the vector ALU reads it and five before a
    memory instruction does, a matrix-core result up to twenty (the longest of the documented cases is
    taken for all), a transcendental result one, and a vector result two before an instruction across
    lanes (DPP, permlane, readlane) or a matrix-core instruction reads it; and the registers that a store of more
    than two dwords sends may be written two wait states behind it.  The compiler puts s_nop between its own
    instructions; a pair of which one is written as asm gets none.  Walks every kernel along all its edges with the least
    number of wait states since each such write, and reports every pair with too few:
    (kernel, line, text, register, wait states there, wait states needed)."""
    rows, kern, in_asm = [], None, False  # labels, kernel starts and instructions with what they read and write
    for i, l in enumerate(open(path)):
        t = l.strip()
        if t.startswith(';;#ASMSTART'): in_asm = True; continue
        if t.startswith(';;#ASMEND'): in_asm = False; continue
        m = re.match(r'^(_Z\w+|\.LBB\w+):', t)
        if m:
            if t[0] == '_': kern = m.group(1)
            rows.append((i, kern, None if t[0] == '_' else m.group(1)))
            continue
        if not kern or not t or t[0] in ';.': continue
        t = t.split(';')[0].strip()
        op = t.split()[0]
        args = [a.split()[0] for a in t[len(op):].split(',') if a.strip()]
        memory = op.startswith(('global_', 'buffer_', 'flat_', 'scratch_', 'ds_'))
        ndst = 0 if 'store' in op or 'write_b' in op else 2 if '_co_' in op or 'v_div_scale' in op or 'swap' in op else 1
        dst = set().union(*[operands(a) for a in args[:ndst]])
        src = set().union(*[operands(a) for a in args[0 if 'swap' in op else ndst:]])
        if op.startswith('v_cmp') and op.endswith('_e32'): dst.add('vcc')
        lanes = op.startswith(('v_readlane', 'v_readfirstlane', 'v_permlane')) or '_dpp' in op
        reader = {}  # wait states that this instruction needs behind each kind of write
        if in_asm and memory: reader = {'sgpr': WAIT_SGPR_MEMORY, 'mfma': WAIT_MFMA}
        elif in_asm and op.startswith('v_'): reader = {'sgpr': WAIT_SGPR_VALU, 'mfma': WAIT_MFMA, 'trans': WAIT_TRANS}
        matrix = op.startswith(('v_mfma', 'v_smfma'))
        if lanes or matrix: reader['asm'] = WAIT_LANES
        writes = []
        if in_asm and memory and 'store' in op and re.search(r'x[34]|b96|b128', op):
            writes += [(r, 'store') for r in operands(args[0 if op.startswith('buffer_') else 1])]
        if op.startswith('v_'):
            for r in dst:
                if r[0] == 's' or r == 'vcc': writes.append((r, 'sgpr'))
                elif matrix: writes.append((r, 'mfma'))
                elif op.startswith(TRANS): writes.append((r, 'trans'))
                elif in_asm: writes.append((r, 'asm'))
        step = int(args[0], 0) + 1 if op == 's_nop' else 1
        rows.append((i, kern, op, t, dst, src, reader, writes, step, args[0] if 'branch' in op else None))
    label_in, found, changed = {}, {}, True
    while changed:  # until the states carried by backward branches settle
        changed, state = False, {}
        for row in rows:
            if len(row) == 3:
                if row[2] is None: state = {}
                for k, n in label_in.get(row[1:], {}).items(): state[k] = min(n, state.get(k, n))
                continue
            i, kern, op, t, dst, src, reader, writes, step, to = row
            for (r, kind), n in state.items():
                if r in src and n < reader.get(kind, 0): found[i] = (kern, i + 1, t, r, n, reader[kind])
                if kind == 'store' and r in dst and op.startswith('v_') and n < WAIT_STORE: found[i] = (kern, i + 1, t, r, n, WAIT_STORE)
            if state:
                state = {k: n + step for k, n in state.items() if n + step < WAIT_MFMA and k[0] not in dst}
            for k in writes: state[k] = 0
            if to:
                at = label_in.setdefault((kern, to), {})
                for k, n in state.items():
                    if n < at.get(k, WAIT_MFMA): at[k] = n; changed = True
            if op in ('s_branch', 's_endpgm', 's_setpc_b64'): state = {}
    return [found[i] for i in sorted(found)]

def report_hazards(bad, limit=40):
    return "\n".join("%s: line %d: '%s' touches %s after %d wait states of %d" % e for e in bad[:limit])

def report(bad, limit=40):
    lines = ["%s: line %d: '%s' %s SGPR %s of the scalar load issued at line %d" % e for e in bad[:limit]]
    return "\n".join(lines)


if __name__ == "__main__":
    bad = scan(sys.argv[1])
    for k, ln, t, what, rr, l0 in bad[:40]:
        print(f"{k}: line {ln}: '{t}' {what} SGPR {rr} of the load issued at line {l0}")
    print("violations:", len(bad))


def kernel_stats(path):
    """Per kernel of a device listing: VGPR spill count from the metadata and how often each
    instruction mnemonic occurs in its body.  Returns {mangled name: (spills, {mnemonic: n})}."""
    import collections
    import re
    body = {}
    name = None
    spills = {}
    cur_meta = None
    for ln in open(path):
        m = re.match(r"^(_Z\w+):", ln)
        if m:
            name = m.group(1)
            body[name] = collections.Counter()
            continue
        t = ln.strip()
        if name and t and not t.startswith((";", ".", "_Z")) and ":" not in t.split()[0]:
            body[name][t.split()[0]] += 1
        if t.startswith(".Lfunc_end"):  # (an early exit's s_endpgm may stand in the middle)
            name = None
        m = re.match(r"^\s+\.name:\s+(\S+)", ln)
        if m:
            cur_meta = m.group(1)
        m = re.match(r"^\s+\.vgpr_spill_count:\s+(\d+)", ln)
        if m and cur_meta:
            spills[cur_meta] = int(m.group(1))
    return {k: (spills.get(k, 0), v) for k, v in body.items() if k in spills}


def metadata(path, field):
    """Per kernel of a device listing: a number of its metadata, e.g. "private_segment_fixed_size" (bytes of
    scratch memory per lane) or "sgpr_spill_count".  Returns {mangled name: number}."""
    out = {}
    text = open(path).read()
    for block in text.split("  - .agpr_count:")[1:]:
        n = re.search(r"\.name:\s+(\S+)", block)
        v = re.search(r"\.%s:\s+(\d+)" % field, block)
        if n and v:
            out[n.group(1)] = int(v.group(1))
    return out
