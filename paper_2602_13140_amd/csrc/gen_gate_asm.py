#!/usr/bin/env python3
"""Writes qsv_gate_asm.h: the text of the inline-assembly gate interpreter of the fused pass
kernel (gfx950).  Run by build.py before hipcc; the header is also committed so that the source
tree compiles as it stands.

Why assembly: the 32 amplitude registers of a lane must stay where they are across the whole
operation list.  A C++ switch over operation kinds makes the compiler copy all of them at every
merge point; one asm block with tied operands and its own scalar dispatch does not.  It also
lets the next operation word and the next matrix be fetched while the current gate computes.

The block executes consecutive operations (2x2 unitary on a register bit, CNOT with the control
in a register bit, CNOT with the control elsewhere in the index or given by the parity of several
index bits, the three forms of CZ sign flips,
and the transpose through LDS that moves the register run) and returns at the first operation of any other kind, leaving the
operation pointer on it and no scalar load or LDS access in flight.

LDS layout: one plane of 2^T floats through which the real parts go first and then the imaginary
parts (the default), or two planes for both at once.  Element tau of a plane sits at index
tau ^ ((tau >> 4) & 31): the XOR spreads every layout's 32 consecutive lanes over the 32 banks,
costs no space, and, XOR being linear, the address of register element k is (lane's part) ^ off(k)
with off(k) the XOR of the offsets of k's set bits.  A layout is therefore described by four
offsets (those of elements 1, 2, 4, 8), kept in vector registers, and the elements are visited in
Gray-code order, so that each address is the previous one XOR one of the four: one vector-only
v_xor per element (a vector instruction with a scalar operand issues at 4.2 cycles per wavefront
on this chip, one with vector operands only at 2.1 to 2.4).
The dynamic LDS segment starts at byte 0 (the kernel has no static LDS), so no base is added.

Operation word: x = kind | a<<8 | b<<16 | c<<24, y = arg.  For a unitary, arg is the index of its
matrix in execution order, so consecutive unitaries read consecutive 32-byte entries and the
next one can be prefetched (the table is padded by one entry for the last prefetch).  An entry is
either the eight floats of the matrix (c = 1) or the matrix without a scalar factor as a rotation
between two phases (c = 0; see rot_pair), whose seventh word picks one of 28 instruction sequences.

Fixed scalar registers (declared as clobbers; the text below names them s52..s56 and s68..s99,
_renumbered() packs them into s36..s72, which leaves the compiler enough of the 96 scalar registers
the kernel is limited to (eight wavefronts per SIMD) to do without spills):
  s[52:55] landing place of a layout's four offsets on their way to vector registers
  s68 layout whose offsets sit in %[ba0..3] (-1: none, the compiler may have used them since)
  s69 one-plane transposes: the exchange crosses wavefronts
  s56 index (in execution order) of the matrix in s[72:79], -1: none; s[70:71] its address
  s[72:79] matrix of the stream: the one in use until its vector copies are made, then the next
  s[80:81] current operation word     s82 kind   s83 field a
  s[84:85] scratch / saved exec       s[86:87] scratch address
  s[88:95] shifted matrix of a gradient row
  s[96:97] operation pointer          s[98:99] next operation word
"""
import os
import re

R = 4
NR = 1 << R
OP_XPOSE, OP_U, OP_CX_REG, OP_CX_DYN, OP_CZ_REG, OP_CZ_MIX, OP_CZ_LANE, OP_CX_CHAIN, OP_CX_PAR, OP_CX_LANE = 2, 3, 4, 5, 6, 7, 8, 9, 10, 12
# the chains of CNOTs between neighbouring register bits, numbered as in the planner:
# (direction, control of the first, count); direction 0: controls go up, 1: down
CX_CHAINS = [(0, 0, 3), (1, 2, 3), (0, 0, 2), (0, 1, 2), (1, 2, 2), (1, 1, 2)]
FIRST_SGPR, LAST_SGPR = 36, 72      # after _renumbered()
GRAY = [i ^ (i >> 1) for i in range(NR)]        # element visited at step i
GRAY_BIT = [0] + [(i & -i).bit_length() - 1 for i in range(1, NR)]   # bit that changes on entering step i


def u_pair(a, b):
    """The product of the pair with a whole matrix (the last unitary of a group, shifted matrices): (r_a,i_a) has the
    target bit 0, (r_b,i_b) has it 1; m0..m7 = vector copies of
    s88..s95 = (m00r, m00i, m01r, m01i, m10r, m10i, m11r, m11i): a vector instruction with a scalar
    operand issues at 4.2 cycles per wavefront on this chip, one with vector operands only at 2.1 to 2.4.
    Four interleaved chains; the last step of each overwrites an input that is dead by then."""
    ra, ia, rb, ib = "%%[r%d]" % a, "%%[i%d]" % a, "%%[r%d]" % b, "%%[i%d]" % b
    t = ["%[t0]", "%[t1]", "%[t2]", "%[t3]"]
    mul = lambda d, m, x: "v_mul_f32 %s, %s, %s" % (d, m, x)
    fma = lambda d, m, x, acc: "v_fma_f32 %s, %s, %s, %s" % (d, m, x, acc)
    return [
        mul(t[0], "%[m0]", ra), mul(t[1], "%[m1]", ra), mul(t[2], "%[m4]", ra), mul(t[3], "%[m5]", ra),
        fma(t[0], "-%[m1]", ia, t[0]), fma(t[1], "%[m0]", ia, t[1]),
        fma(t[2], "-%[m5]", ia, t[2]), fma(t[3], "%[m4]", ia, t[3]),
        fma(t[0], "%[m2]", rb, t[0]), fma(t[1], "%[m3]", rb, t[1]),
        fma(t[2], "%[m6]", rb, t[2]), fma(t[3], "%[m7]", rb, t[3]),
        fma(ra, "-%[m3]", ib, t[0]), fma(ia, "%[m2]", ib, t[1]),
        fma(rb, "-%[m7]", ib, t[2]), fma(ib, "%[m6]", ib, t[3]),
    ]


# Forms of a factored unitary: which phases it has, and its core.  With both phases, A and B after the name say
# that the one before or after the core has a quarter turn taken out of it.
FORMS = ("none", "before", "after", "both", "bothA", "bothB", "bothAB")
CORES = ("c+", "c-", "s+", "s-")
ROT_LENGTH = {"none": 6, "before": 7, "after": 7, "both": 10, "bothA": 10, "bothB": 10, "bothAB": 10}


def rot_pair(a, b, form, core):
    """A unitary without its scalar factor, on the pair p (target bit 0) and q (target bit 1):
    diag(1, e^iB) core diag(1, e^iA) with |A|, |B| <= pi/2 (both phases: diag(1, i^b e^iB) core diag(1, i^a e^iA) with
    |A|, |B| <= pi/4 and a, b as the form says).  The cores are the real rotations divided by
    their larger entry,
      c+- : p' = p + x q,     q' = y p +- q          s+- : p' = x p -+ q,    q' = p + y q,     |x|, |y| <= 1,
    so each of the four real results takes one multiply-add.  A phase turns (re, im) of q by three shears
    re += t im, im += s re, re += t im with t = -tan(A/2), s = sin A, in place.  4 + 3 (+ 3)
    instructions where the matrix product takes 12 (14): the unitaries are 80 % of a pass's vector
    instructions, and vector issue bounds the passes.
    The quarter turns cost no instruction (registers change names and signs).  Without them the larger t and s of
    the larger angles, and the larger numbers between the shears, made unitaries with two phases round worse than the
    matrix product: RX RY on 16 qubits, 20 layers 9.7e-7 against 8.1e-7 from 64 bits.
    Entry: m0, m1 = t, s of A; m2, m3 = x, y; m4, m5 = t, s of B."""
    ra, ia, rb, ib = "%%[r%d]" % a, "%%[i%d]" % a, "%%[r%d]" % b, "%%[i%d]" % b
    t0, t1 = "%[t0]", "%[t1]"
    m = ["%%[m%d]" % k for k in range(6)]
    neg = lambda r: r[1:] if r[0] == "-" else "-" + r

    def fma(d, f, v, acc):
        if d == acc and "-" not in (f + v):
            return "v_fmac_f32 %s, %s, %s" % (d, f, v)
        return "v_fma_f32 %s, %s, %s, %s" % (d, f, v, acc)

    minus = core[1] == "-"
    out = []
    if form == "none":                     # q' waits in temporaries until p' has read q
        qr, qi, nr, ni = rb, ib, t0, t1
    elif form == "before":                 # the turned q sits in temporaries, q' goes to its place
        out += [fma(t0, m[0], ib, rb), fma(t1, m[1], t0, ib), fma(t0, m[0], t1, t0)]
        qr, qi, nr, ni = t0, t1, rb, ib
    elif form == "after":                  # q' in temporaries, the shears bring it home
        qr, qi, nr, ni = rb, ib, t0, t1
    else:
        out += [fma(t0, m[0], ib, rb), fma(t1, m[1], t0, ib), fma(t0, m[0], t1, t0)]
        qr, qi, nr, ni = t0, t1, rb, ib
        if "A" in form:                    # i q
            qr, qi = neg(t1), t0
        if "B" in form:                    # q' goes to the place of i q'
            nr, ni = ib, neg(rb)

    def to(d, f, v, acc):                  # d may be the negative of a register
        return fma(d, f, v, acc) if d[0] != "-" else fma(d[1:], neg(f), v, neg(acc))

    if core[0] == "c":
        out += [to(nr, m[3], ra, neg(qr) if minus else qr), to(ni, m[3], ia, neg(qi) if minus else qi),
                fma(ra, m[2], qr, ra), fma(ia, m[2], qi, ia)]
    else:
        out += [to(nr, m[3], qr, ra), to(ni, m[3], qi, ia),
                fma(ra, m[2], ra, qr if minus else neg(qr)), fma(ia, m[2], ia, qi if minus else neg(qi))]
    if form == "none":
        out += ["v_mov_b32 %s, %s" % (rb, t0), "v_mov_b32 %s, %s" % (ib, t1)]
    elif form == "after":
        out += [fma(rb, m[4], t1, t0), fma(ib, m[5], rb, t1), fma(rb, m[4], ib, rb)]
    elif form.startswith("both"):
        out += [fma(rb, m[4], ib, rb), fma(ib, m[5], rb, ib), fma(rb, m[4], ib, rb)]
    return out


CHAIN_FORM = "move"     # "swap": every cycle by v_swap_b32


def chain_swaps(direction, first, count):
    """The chain's CNOTs (control c, target c + 1) as one permutation of the 16 register elements.  A cycle of
    k elements takes k - 1 swaps (v_swap_b32, 8.2 cycles each) or k + 1 moves through a temporary (2.1 to 2.4
    cycles each): cycles of two are swapped, longer ones moved.  Measured on one box, alternating the two
    builds: moves take 0.8 % off the 26-qubit and 20-qubit configurations now that their passes are
    heavy (when the passes were lighter and waited for memory the same change cost 0.6 %)."""
    src = list(range(NR))                  # src[i]: which old element ends up in place i
    for k in range(count):
        c = first + k if direction == 0 else first - k
        t = c + 1
        for i in range(NR):
            if (i >> c) & 1 and not (i >> t) & 1:
                j = i | (1 << t)
                src[i], src[j] = src[j], src[i]
    out, seen = [], [False] * NR
    for s0 in range(NR):
        if seen[s0] or src[s0] == s0:
            continue
        cyc, cur = [], s0
        while not seen[cur]:
            seen[cur] = True
            cyc.append(cur)
            cur = src[cur]
        if CHAIN_FORM == "move" and len(cyc) > 2:
            # place cyc[k] receives the old content of cyc[k+1]; the first one's goes round through a temporary
            for part, tmp in (("r", "%[t0]"), ("i", "%[t1]")):
                reg = lambda k: "%%[%s%d]" % (part, k)
                out.append("v_mov_b32 %s, %s" % (tmp, reg(cyc[0])))
                for a, b in zip(cyc, cyc[1:]):
                    out.append("v_mov_b32 %s, %s" % (reg(a), reg(b)))
                out.append("v_mov_b32 %s, %s" % (reg(cyc[-1]), tmp))
            continue
        # place cyc[k] must receive the old content of cyc[k+1]: swap neighbours along the cycle
        for a, b in zip(cyc, cyc[1:]):
            out.extend(swap_pair(a, b))
    return out


def swap_pair(a, b):
    return ["v_swap_b32 %%[r%d], %%[r%d]" % (a, b), "v_swap_b32 %%[i%d], %%[i%d]" % (a, b)]


def gen(planes=2, perlane=False):
    """perlane: the variant for kernels whose tiles hold several state rows, where a unitary whose
    matrix depends on the row is left to the caller."""
    assert planes in (1, 2)
    L = []
    emit = L.append
    lab = lambda name: "L_%s_%%=" % name
    ALIGN = ".p2align 6"                          # branch targets start an instruction-fetch line

    def prefetch_next_word():
        emit("s_load_dwordx2 s[98:99], s[96:97], 0x8")

    emit("s_mov_b32 s96, %[opslo]")
    emit("s_mov_b32 s97, %[opshi]")
    emit("s_mov_b32 s56, -1")                     # no matrix prefetched yet
    emit("s_mov_b32 s68, -1")
    emit("s_load_dwordx2 s[98:99], s[96:97], 0x0")
    emit("s_branch " + lab("top"))
    emit(ALIGN)
    emit(lab("next") + ":")                       # falls through to the top: one jump per operation
    emit("s_add_u32 s96, s96, 8")
    emit("s_addc_u32 s97, s97, 0")
    emit(lab("top") + ":")
    emit("s_waitcnt lgkmcnt(0)")                  # next word and prefetched matrix have landed
    emit("s_mov_b64 s[80:81], s[98:99]")
    emit("s_and_b32 s82, s80, 0xff")
    emit("s_bfe_u32 s83, s80, 0x80008")
    emit("s_cmp_eq_u32 s82, %d" % OP_U)
    emit("s_cbranch_scc1 " + lab("u"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CX_CHAIN)
    emit("s_cbranch_scc1 " + lab("cxc"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CX_REG)
    emit("s_cbranch_scc1 " + lab("cxr"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CX_DYN)
    emit("s_cbranch_scc1 " + lab("cxd"))
    emit("s_cmp_eq_u32 s82, %d" % OP_XPOSE)
    emit("s_cbranch_scc1 " + lab("xp"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CX_LANE)
    emit("s_cbranch_scc1 " + lab("cxl"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CX_PAR)
    emit("s_cbranch_scc1 " + lab("cxp"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CZ_REG)
    emit("s_cbranch_scc1 " + lab("zr"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CZ_MIX)
    emit("s_cbranch_scc1 " + lab("zm"))
    emit("s_cmp_eq_u32 s82, %d" % OP_CZ_LANE)
    emit("s_cbranch_scc1 " + lab("zl"))
    emit("s_branch " + lab("exit"))

    # ---- 2x2 unitary on register bit a; matrix = (arg == ovrid) ? *ovr : mbase[arg].
    # s[72:79] holds the matrix of the stream with index s56 (-1: none), s[70:71] its address; the
    # multiply sequences read vector copies, so the buffer is free for the next matrix of the stream
    # as soon as the copies are made.  Every scalar instruction here competes with the vector ones
    # for issue slots, hence the short common path: three tests and one computed jump.
    emit(ALIGN)
    emit(lab("u") + ":")
    if perlane:
        emit("s_bfe_u32 s84, s80, 0x80010")      # b: matrix depends on the state row
        emit("s_and_b32 s84, s84, %[nonuni]")    # ... and rows differ per lane: not ours
        emit("s_cmp_lg_u32 s84, 0")
        emit("s_cbranch_scc1 " + lab("exit"))
    emit("s_cmp_eq_u32 s81, %[ovrid]")
    emit("s_cbranch_scc1 " + lab("uovr"))
    emit("s_cmp_eq_u32 s81, s56")
    emit("s_cbranch_scc0 " + lab("uld"))
    emit(lab("uhave") + ":")
    emit("s_bitcmp1_b32 s80, 24")                 # c: the entry is the matrix itself
    emit("s_cbranch_scc1 " + lab("ug"))
    # factored: jump through a table of branches, 4 * (4 * sequence + register bit) bytes into it
    emit("s_lshl_b32 s84, s83, 2")
    emit("s_add_u32 s84, s84, s78")
    emit("s_add_u32 s84, s84, 12")                # the three instructions before the table
    emit("s_getpc_b64 s[86:87]")
    emit("s_add_u32 s86, s86, s84")
    emit("s_addc_u32 s87, s87, 0")
    emit("s_setpc_b64 s[86:87]")
    for form in FORMS:
        for core in range(len(CORES)):
            for j in range(R):
                emit("s_branch " + lab("r%s%d%d" % (form, core, j)))

    def stream_next():
        emit("s_add_u32 s70, s70, 32")            # prefetch the next entry of the stream
        emit("s_addc_u32 s71, s71, 0")
        emit("s_add_u32 s56, s56, 1")
        emit("s_load_dwordx8 s[72:79], s[70:71], 0x0")

    for form in FORMS:
        for core, name in enumerate(CORES):
            used = sorted({int(m) for ln in rot_pair(0, 1, form, name) for m in re.findall(r"%\[m(\d)\]", ln)})
            for j in range(R):
                emit(ALIGN)
                emit(lab("r%s%d%d" % (form, core, j)) + ":")
                for k in used:                    # the sequences read vector registers only
                    emit("v_mov_b32 %%[m%d], s%d" % (k, 72 + k))
                stream_next()
                prefetch_next_word()
                for i in range(NR):
                    if not i & (1 << j):
                        L.extend(rot_pair(i, i | (1 << j), form, name))
                emit("s_branch " + lab("next"))
    emit(ALIGN)
    emit(lab("ug") + ":")
    for k in range(8):
        emit("v_mov_b32 %%[m%d], s%d" % (k, 72 + k))
    stream_next()
    emit(lab("ugj") + ":")                        # the shifted matrix of a gradient row joins here
    prefetch_next_word()
    for j in range(R - 1):
        emit("s_cmp_eq_u32 s83, %d" % j)
        emit("s_cbranch_scc1 " + lab("ug%d" % j))
    for j in reversed(range(R)):
        emit(ALIGN)
        emit(lab("ug%d" % j) + ":")
        for i in range(NR):
            if not i & (1 << j):
                L.extend(u_pair(i, i | (1 << j)))
        emit("s_branch " + lab("next"))
    # not the prefetched one (first unitary of a tile, or the one after a shifted matrix): fetch it
    emit(lab("uld") + ":")
    emit("s_lshl_b32 s84, s81, 5")
    emit("s_add_u32 s70, %[mlo], s84")
    emit("s_addc_u32 s71, %[mhi], 0")
    emit("s_mov_b32 s56, s81")
    emit("s_load_dwordx8 s[72:79], s[70:71], 0x0")
    emit("s_waitcnt lgkmcnt(0)")
    emit("s_branch " + lab("uhave"))
    # the shifted matrix of a gradient row: not part of the stream, general multiply sequence
    emit(lab("uovr") + ":")
    emit("s_mov_b32 s86, %[olo]")
    emit("s_mov_b32 s87, %[ohi]")
    emit("s_load_dwordx8 s[88:95], s[86:87], 0x0")
    emit("s_waitcnt lgkmcnt(0)")
    for k in range(8):
        emit("v_mov_b32 %%[m%d], s%d" % (k, 88 + k))
    emit("s_branch " + lab("ugj"))

    # ---- CNOT, control = register bit b, target = register bit a
    emit(ALIGN)
    emit(lab("cxr") + ":")
    prefetch_next_word()
    emit("s_bfe_u32 s84, s80, 0x80010")
    emit("s_lshl_b32 s85, s83, 2")
    emit("s_add_u32 s84, s84, s85")
    # searched in this order: first the neighbours a CNOT ring produces (target just above the
    # control), since every compare is an instruction that competes with the vector ones for issue
    combos = [(jc + 1, jc) for jc in range(R - 1)]
    combos += [(jt, jc) for jt in range(R) for jc in range(R) if jt != jc and (jt, jc) not in combos]
    for jt, jc in combos:
        emit("s_cmp_eq_u32 s84, %d" % (jt * 4 + jc))
        emit("s_cbranch_scc1 " + lab("x%d%d" % (jt, jc)))
    emit("s_branch " + lab("next"))               # unknown combination: no-op (never planned)
    for jt, jc in combos:
        emit(ALIGN)
        emit(lab("x%d%d" % (jt, jc)) + ":")
        for i in range(NR):
            if (i & (1 << jc)) and not (i & (1 << jt)):
                L.extend(swap_pair(i, i | (1 << jt)))
        emit("s_branch " + lab("next"))

    # ---- chain of CNOTs between neighbouring register bits: arg numbers the chain
    emit(ALIGN)
    emit(lab("cxc") + ":")
    prefetch_next_word()
    for k in range(len(CX_CHAINS) - 1):
        emit("s_cmp_eq_u32 s81, %d" % k)
        emit("s_cbranch_scc1 " + lab("c%d" % k))
    for k in reversed(range(len(CX_CHAINS))):
        emit(ALIGN)
        emit(lab("c%d" % k) + ":")
        L.extend(chain_swaps(*CX_CHAINS[k]))
        emit("s_branch " + lab("next"))

    # ---- CNOT, control = index bit b outside the register run (lane-dependent), target = a
    emit(ALIGN)
    emit(lab("cxd") + ":")
    prefetch_next_word()
    emit("s_bfe_u32 s86, s80, 0x80010")
    emit("s_lshl_b64 s[84:85], 1, s86")
    emit("v_and_b32 %[tc], s84, %[e0lo]")
    emit("v_and_b32 %[t0], s85, %[e0hi]")
    emit("v_or_b32 %[tc], %[tc], %[t0]")
    emit("v_cmp_ne_u32 vcc, 0, %[tc]")
    emit(lab("cxdx") + ":")
    emit("s_and_saveexec_b64 s[84:85], vcc")
    emit("s_cbranch_execz " + lab("cxdone"))
    for j in range(R - 1):
        emit("s_cmp_eq_u32 s83, %d" % j)
        emit("s_cbranch_scc1 " + lab("d%d" % j))
    for j in reversed(range(R)):
        emit(ALIGN)
        emit(lab("d%d" % j) + ":")
        for i in range(NR):
            if not (i & (1 << j)):
                L.extend(swap_pair(i, i | (1 << j)))
        if j != 0:
            emit("s_branch " + lab("cxdone"))
    emit(lab("cxdone") + ":")
    emit("s_mov_b64 exec, s[84:85]")
    emit("s_branch " + lab("next"))

    # ---- CNOT, target = register bit a, control = parity of the lane's index bits in arg (a mask
    # over the low 32 bits of the extended index, none of them in the register run): the condition,
    # then the swaps of the handler above
    emit(ALIGN)
    emit(lab("cxp") + ":")
    prefetch_next_word()
    emit("v_and_b32 %[tc], s81, %[e0lo]")
    emit("v_bcnt_u32_b32 %[tc], %[tc], 0")
    emit("v_and_b32 %[tc], 1, %[tc]")
    emit("v_cmp_ne_u32 vcc, 0, %[tc]")
    emit("s_branch " + lab("cxdx"))



    # ---- CNOT, control = register bit a, target = bit b of the lane number: every lane trades its
    # eight amplitudes with the control set for the partner lane's (lane ^ 2^b).  b = 0, 1: DPP
    # quad permutes, in place; b >= 2: ds_bpermute_b32 (lane crossbar of the LDS unit, no memory
    # involved) with the partner's byte address in %[tc].
    emit(ALIGN)
    emit(lab("cxl") + ":")
    prefetch_next_word()
    emit("s_bfe_u32 s84, s80, 0x80010")           # b
    emit("s_cmp_eq_u32 s84, 0")
    emit("s_cbranch_scc1 " + lab("cxlq0"))
    emit("s_cmp_eq_u32 s84, 1")
    emit("s_cbranch_scc1 " + lab("cxlq1"))
    emit("s_lshl_b32 s85, 1, s84")
    emit("v_xor_b32 %[tc], s85, %[thr]")
    emit("v_and_b32 %[tc], 63, %[tc]")
    emit("v_lshlrev_b32 %[tc], 2, %[tc]")
    for j in range(R - 1):
        emit("s_cmp_eq_u32 s83, %d" % j)
        emit("s_cbranch_scc1 " + lab("cxlb%d" % j))
    for j in reversed(range(R)):
        emit(ALIGN)
        emit(lab("cxlb%d" % j) + ":")
        for k in range(NR):
            if (k >> j) & 1:
                emit("ds_bpermute_b32 %%[r%d], %%[tc], %%[r%d]" % (k, k))
                emit("ds_bpermute_b32 %%[i%d], %%[tc], %%[i%d]" % (k, k))
        emit("s_branch " + lab("next"))           # the wait at the top covers the exchange
    for b, perm in ((0, "[1,0,3,2]"), (1, "[2,3,0,1]")):
        emit(lab("cxlq%d" % b) + ":")
        for j in range(R - 1):
            emit("s_cmp_eq_u32 s83, %d" % j)
            emit("s_cbranch_scc1 " + lab("cxlq%d_%d" % (b, j)))
        for j in reversed(range(R)):
            emit(ALIGN)
            emit(lab("cxlq%d_%d" % (b, j)) + ":")
            for k in range(NR):
                if (k >> j) & 1:
                    for part in "ri":
                        emit("v_mov_b32_dpp %%[%s%d], %%[%s%d] quad_perm:%s row_mask:0xf bank_mask:0xf"
                             % (part, k, part, k, perm))
            emit("s_branch " + lab("next"))

    def flip(part, k):
        return "v_xor_b32 %%[%s%d], 0x80000000, %%[%s%d]" % (part, k, part, k)

    # ---- CZ between register bits a < b: the amplitudes with both bits set change sign
    emit(ALIGN)
    emit(lab("zr") + ":")
    prefetch_next_word()
    emit("s_bfe_u32 s84, s80, 0x80010")
    emit("s_lshl_b32 s85, s83, 2")
    emit("s_add_u32 s84, s84, s85")
    pairs = [(ja, jb) for ja in range(R) for jb in range(ja + 1, R)]
    for ja, jb in pairs:
        emit("s_cmp_eq_u32 s84, %d" % (ja * 4 + jb))
        emit("s_cbranch_scc1 " + lab("zr%d%d" % (ja, jb)))
    emit("s_branch " + lab("next"))               # unknown combination: no-op (never planned)
    for ja, jb in pairs:
        emit(lab("zr%d%d" % (ja, jb)) + ":")
        for k in range(NR):
            if (k >> ja) & 1 and (k >> jb) & 1:
                emit(flip("r", k))
                emit(flip("i", k))
        emit("s_branch " + lab("next"))

    # ---- CZ between register bit a and index bit b outside the run: lanes whose bit b is set
    # flip the sign of the amplitudes with register bit a set
    emit(ALIGN)
    emit(lab("zm") + ":")
    prefetch_next_word()
    emit("s_bfe_u32 s86, s80, 0x80010")
    emit("s_lshl_b64 s[84:85], 1, s86")
    emit("v_and_b32 %[tc], s84, %[e0lo]")
    emit("v_and_b32 %[t0], s85, %[e0hi]")
    emit("v_or_b32 %[tc], %[tc], %[t0]")
    emit("v_cmp_ne_u32 vcc, 0, %[tc]")
    emit("s_and_saveexec_b64 s[84:85], vcc")
    emit("s_cbranch_execz " + lab("zdone"))
    for j in range(R - 1):
        emit("s_cmp_eq_u32 s83, %d" % j)
        emit("s_cbranch_scc1 " + lab("zm%d" % j))
    for j in reversed(range(R)):
        emit(lab("zm%d" % j) + ":")
        for k in range(NR):
            if (k >> j) & 1:
                emit(flip("r", k))
                emit(flip("i", k))
        emit("s_branch " + lab("zdone"))

    # ---- CZ rungs (mask in arg, bit q = rung (q, q+1)) between index bits outside the run: one
    # sign per lane, parity of popcount(e0 & (e0 >> 1) & mask); the mask lies below bit 31
    emit(ALIGN)
    emit(lab("zl") + ":")
    prefetch_next_word()
    emit("v_lshrrev_b32 %[t0], 1, %[e0lo]")
    emit("v_and_b32 %[t0], %[t0], %[e0lo]")
    emit("v_and_b32 %[t0], s81, %[t0]")
    emit("v_bcnt_u32_b32 %[t0], %[t0], 0")
    emit("v_and_b32 %[t0], 1, %[t0]")
    emit("v_cmp_ne_u32 vcc, 0, %[t0]")
    emit("s_and_saveexec_b64 s[84:85], vcc")
    emit("s_cbranch_execz " + lab("zdone"))
    for k in range(NR):
        emit(flip("r", k))
        emit(flip("i", k))
    emit(lab("zdone") + ":")
    emit("s_mov_b64 exec, s[84:85]")
    emit("s_branch " + lab("next"))

    # ---- transpose: move the register run from layout scur to layout a (field a of the word).
    # The four address offsets of a layout come from a 4-dword table row (one scalar load) and go to
    # vector registers: %[ba0..3] for the layout named in s68 (-1: none), %[bb0..3] for the layout
    # being moved to.
    def load_offsets(sreg):
        emit("s_lshl_b32 s84, %s, 4" % sreg)
        emit("s_add_u32 s86, %[tablo], s84")
        emit("s_addc_u32 s87, %[tabhi], 0")
        emit("s_load_dwordx4 s[52:55], s[86:87], 0x0")

    def offsets_to(prefix):
        for j in range(4):
            emit("v_mov_b32 %%[%s%d], s%d" % (prefix, j, 52 + j))

    tmps = ["%[t0]", "%[t1]", "%[t2]", "%[t3]"]

    def walk(base, prefix, access):
        """Visits the 16 register elements in Gray-code order; access(k, address register)."""
        prev = base
        for i in range(NR):
            if i:
                t = tmps[i % 4]
                emit("v_xor_b32 %s, %s, %%[%s%d]" % (t, prev, prefix, GRAY_BIT[i]))
                prev = t
            access(GRAY[i], prev)

    def lane_part(dst):
        """dst = byte address part of the lane in layout scur; also refreshes e0."""
        # tau = ((thr >> s) << (s + 4)) | (thr & ((1 << s) - 1))
        emit("v_lshrrev_b32 %[t0], %[scur], %[thr]")
        emit("s_add_u32 s84, %[scur], 4")
        emit("v_lshlrev_b32 %[t0], s84, %[t0]")
        emit("s_lshl_b32 s85, 1, %[scur]")
        emit("s_sub_u32 s85, s85, 1")
        emit("v_and_b32 %[t1], s85, %[thr]")
        emit("v_or_b32 %[t0], %[t0], %[t1]")          # t0 = tau of the lane (register bits zero)
        emit("v_lshrrev_b32 %[t1], 4, %[t0]")
        emit("v_and_b32 %[t1], 31, %[t1]")
        emit("v_xor_b32 %[t1], %[t1], %[t0]")
        emit("v_lshlrev_b32 " + dst + ", 2, %[t1]")   # swz(tau) * 4
        # extended index of the lane: e0 = tile_base | (tau & cmask) | ((tau >> c) << w), w < 32
        emit("v_lshrrev_b32 %[t1], %[c], %[t0]")
        emit("v_and_b32 %[t2], %[cmask], %[t0]")
        emit("v_lshlrev_b32 %[t3], %[w], %[t1]")
        emit("v_or_b32 %[t2], %[t2], %[t3]")
        emit("v_or_b32 %[e0lo], %[tblo], %[t2]")
        emit("s_sub_u32 s84, 32, %[w]")
        emit("v_lshrrev_b32 %[t1], s84, %[t1]")
        emit("v_or_b32 %[e0hi], %[tbhi], %[t1]")

    emit(ALIGN)
    emit(lab("xp") + ":")
    prefetch_next_word()
    emit("s_cmp_eq_u32 s68, %[scur]")
    emit("s_cbranch_scc1 " + lab("xphave"))
    load_offsets("%[scur]")
    emit("s_waitcnt lgkmcnt(0)")
    offsets_to("ba")
    emit(lab("xphave") + ":")
    emit("s_bfe_u32 s84, s80, 0x80018")           # c: barrier before the writes
    emit("s_cmp_eq_u32 s84, 0")
    emit("s_cbranch_scc1 " + lab("xpw"))
    emit("s_barrier")
    emit(lab("xpw") + ":")
    if planes == 2:
        walk("%[ldsb]", "ba", lambda k, t: emit(
            "ds_write2st64_b32 %s, %%[r%d], %%[i%d] offset1:%%[pl64]" % (t, k, k)))
        # new layout: its offsets first (they arrive while the lane's own part is computed)
        emit("s_mov_b32 %[scur], s83")
        load_offsets("%[scur]")
        lane_part("%[ldsb]")
        emit("s_waitcnt lgkmcnt(0)")              # own writes are in LDS, new offsets are here
        offsets_to("ba")
        emit("s_mov_b32 s68, %[scur]")
        emit("s_bfe_u32 s84, s80, 0x80010")       # b: the exchange crosses wavefronts
        emit("s_cmp_eq_u32 s84, 0")
        emit("s_cbranch_scc1 " + lab("xpr"))
        emit("s_barrier")
        emit(lab("xpr") + ":")

        def read2(k, t):
            emit("ds_read_b32 %%[r%d], %s" % (k, t))
            emit("ds_read_b32 %%[i%d], %s offset:%%[plane4]" % (k, t))
        walk("%[ldsb]", "ba", read2)
        emit("s_branch " + lab("next"))           # the wait at the top covers the reads
    else:
        # One plane: real parts go through it first, then the imaginary parts.  The offsets of the
        # new layout sit in %[bb0..3] until the end, the lane's new address part in ldsn.  A
        # wavefront's LDS operations execute in order, so the steps need a wait and a barrier
        # between them only when the exchange crosses wavefronts (flag b, kept in s69).
        def sync(name):
            emit("s_cmp_eq_u32 s69, 0")
            emit("s_cbranch_scc1 " + lab(name))
            emit("s_waitcnt lgkmcnt(0)")
            emit("s_barrier")
            emit(lab(name) + ":")

        def writes(part):
            walk("%[ldsb]", "ba", lambda k, t: emit("ds_write_b32 %s, %%[%s%d]" % (t, part, k)))

        def reads(part):
            walk("%[ldsn]", "bb", lambda k, t: emit("ds_read_b32 %%[%s%d], %s" % (part, k, t)))

        emit("s_bfe_u32 s69, s80, 0x80010")
        writes("r")
        emit("s_mov_b32 %[scur], s83")
        load_offsets("%[scur]")
        lane_part("%[ldsn]")
        emit("s_waitcnt lgkmcnt(0)")              # new offsets are here (and own writes landed)
        offsets_to("bb")
        emit("s_cmp_eq_u32 s69, 0")
        emit("s_cbranch_scc1 " + lab("xpr"))
        emit("s_barrier")
        emit(lab("xpr") + ":")
        reads("r")
        sync("xpw2")
        writes("i")
        sync("xpr2")
        reads("i")
        for j in range(4):                        # the new layout's offsets become the current ones
            emit("v_mov_b32 %%[ba%d], %%[bb%d]" % (j, j))
        emit("s_mov_b32 s68, %[scur]")
        emit("v_mov_b32 %[ldsb], %[ldsn]")
        emit("s_branch " + lab("next"))           # the wait at the top covers the reads

    emit(lab("exit") + ":")                       # reached right after the wait: nothing in flight
    emit("s_mov_b32 %[opslo], s96")
    emit("s_mov_b32 %[opshi], s97")
    return [_renumbered(ln) for ln in L]


def _renumbered(line):
    """Packs the block's scalar registers: s52..s55 -> s36..s39, s68..s99 -> s40..s71 (both shifts
    keep the alignment that register pairs, quads and octets need), s56 -> s72."""
    import re

    def new(n):
        n = int(n)
        if 52 <= n <= 55:
            return n - 16
        if n == 56:
            return 72
        assert 68 <= n <= 99, n
        return n - 28
    line = re.sub(r"\bs\[(\d+):(\d+)\]", lambda m: "s[%d:%d]" % (new(m.group(1)), new(m.group(2))), line)
    return re.sub(r"\bs(\d+)\b", lambda m: "s%d" % new(m.group(1)), line)


# ==================================================================================================
# The direct interpreter: the form of the block for tiles of one state row (see k_pass_direct).
#
# Measured with eight wavefronts per SIMD: a vector instruction on vector registers takes 2.1 to 2.4
# cycles of its SIMD, one with a scalar source 4, v_swap_b32 8, a scalar instruction 4 (beside the vector
# ones, up to one for two of them).  The interpreter above spends 28 scalar instructions on a
# unitary of 56 to 80 vector ones, 20 to 40 on a gate of 8 to 16, and 95 vector instructions on a
# transpose that only moves data; a shift-rule pass issued 0.6 scalar instructions per vector one.  Here
#   - an operation word holds the offset of its code (low half; the host knows where every
#     sequence starts) and its argument (high half): a wait, two additions and a jump per operation,
#   - the table entries of the unitaries are read strictly in order, so there is no index to compare, and
#     an entry holds the offset of its sequence,
#   - every register layout has its own transpose code, with the elements at immediate offsets: element tau
#     of the plane sits at tau + 2 (tau >> 5), which is additive over disjoint bits, so an element's
#     address is the lane's part plus a constant.  The two words of padding per 32 keep 32 consecutive
#     lanes on 32 banks in every layout but 0 (there two lanes share a bank),
#   - exchanges of registers are moves (three of 2.1 cycles) instead of swaps.
#
# Fixed scalar registers:
#   s[36:37] address of the block's first instruction (code offsets count from it)
#   s[38:39] operation list   s40 byte offset of the next word   s[42:43] the word (code, argument)
#   s[44:45] matrix table     s41 byte offset of the next entry   s[48:55] the next entry
#   s[56:63] shifted matrix of a gradient row
#   s[64:65], s[66:67] jump targets   s[68:69] saved exec   s70 argument of a transpose or a turn
#
# The paired form (pair=True) is the same block for two states at once, psi in r, i and lambda in p, q: the reverse-mode
# sweep takes both back through a pass and reads the transition sums off the registers between the gates (see
# sum_handlers).  Every operation acts on psi first and then on lambda, with one fetch, one dispatch and one set of
# numbers for both; a transpose moves four parts through the plane.  It has no whole or shifted matrices, keeps what waits
# in t2, t3 and tc of the single form in registers that are free then (80 registers in all: six wavefronts per SIMD), and uses besides
#   s[72:73] where the next record of sums goes   s[74:75] lanes 0, 16, 32 and 48
DIRECT_FIRST, DIRECT_LAST, PAIR_LAST = 36, 70, 75
LAYOUTS = 11                                     # register runs at tile bits 0..10


def u_stride(pair):
    """Bytes from one register bit's code of a unitary to the next one's."""
    return 1088 if pair else 576


X_DELTA = LAYOUTS * 256                          # bytes from a layout's code for one of a transpose's parts to the next one's
PARTS = (("", "r"), ("I", "i"), ("L", "p"), ("LI", "q"))


CZ_RUNGS = 3                                     # rungs between neighbouring register bits
OVERRIDE_NONE = 0xffffffff


def padded(tau):
    return tau + 2 * (tau >> 5)


def size_of(line):
    """Bytes of one of the instructions used here."""
    op = line.split()[0]
    if op.startswith(("v_fma_", "ds_", "s_load_", "global_")) or op in ("v_lshl_or_b32", "v_lshl_add_u32", "v_bcnt_u32_b32"):
        return 8
    if op.endswith("_dpp"):
        return 8
    literal = re.search(r"(?:^|[ ,])(0x[0-9a-f]+|\d+)\s*(?:,|$)", line.split(None, 1)[1]) if " " in line else None
    if literal and not op.startswith(("s_waitcnt", "s_cbranch", "s_branch", "s_bitcmp", "s_nop")) and int(literal.group(1), 0) > 64:
        return 8
    return 4


def move_pairs(pairs):
    """Exchanges register elements: three moves through a temporary each."""
    out = []
    for a, b in pairs:
        for part, tmp in (("r", "%[t0]"), ("i", "%[t1]")):
            ra, rb = "%%[%s%d]" % (part, a), "%%[%s%d]" % (part, b)
            out += ["v_mov_b32 %s, %s" % (tmp, ra), "v_mov_b32 %s, %s" % (ra, rb), "v_mov_b32 %s, %s" % (rb, tmp)]
    return out


def chain_moves(direction, first, count):
    """chain_swaps with its exchanges of two as moves as well."""
    out = []
    for ln in chain_swaps(direction, first, count):
        m = re.match(r"v_swap_b32 (%\[[ri]\d+\]), (%\[[ri]\d+\])", ln)
        if m:
            out += ["v_mov_b32 %%[t0], %s" % m.group(1), "v_mov_b32 %s, %s" % m.groups(),
                    "v_mov_b32 %s, %%[t0]" % m.group(2)]
        else:
            out.append(ln)
    return out


def cz_elements(mask):
    """Register elements whose sign the rungs of mask (bit j: between register bits j and j + 1) flip."""
    return [k for k in range(NR) if bin(k & (k >> 1) & mask).count("1") & 1]


NEXT_WORD = ["s_add_u32 s40, s40, 8", "s_load_dwordx2 s[42:43], s[38:39], s40"]
NEXT_ENTRY = ["s_add_u32 s41, s41, 32", "s_load_dwordx8 s[48:55], s[44:45], s41"]
DISPATCH = ["s_waitcnt lgkmcnt(0)",              # the next word and entry have landed, and what LDS owes
            "s_add_u32 s64, s36, s42", "s_addc_u32 s65, s37, 0", "s_setpc_b64 s[64:65]"]


def of_lambda(lines):
    """Lines that work on psi's registers, on lambda's."""
    return [re.sub(r"%\[([ri])(\d+)\]", lambda m: "%%[%s%s]" % ("p" if m.group(1) == "r" else "q", m.group(2)), ln)
            for ln in lines]


AXES = "XYZ"


def sum_terms(axis, a, b):
    """Im <lambda| P |psi> of one pair, P the Pauli matrix of the axis, as (sign, lambda's, psi's register), the first
    with a plus sign."""
    ra, ia, rb, ib = ("%%[%s%d]" % (x, k) for k in (a, b) for x in "ri")
    pa, qa, pb, qb = ("%%[%s%d]" % (x, k) for k in (a, b) for x in "pq")
    return {"X": [(1, pa, ib), (-1, qa, rb), (1, pb, ia), (-1, qb, ra)],
            "Y": [(1, pb, ra), (1, qb, ia), (-1, pa, rb), (-1, qa, ib)],
            "Z": [(1, pa, ia), (-1, qa, ra), (-1, pb, ib), (1, qb, rb)]}[axis]


def lane_sums(j, axes, accs):
    """The sums of the lane's eight pairs of register bit j, one axis into each of accs: four multiply-adds a pair."""
    out, fresh = [], set(accs)
    for i in range(NR):
        if not i & (1 << j):
            for rank in range(4):
                for axis, acc in zip(axes, accs):
                    sign, x, y = sum_terms(axis, i, i | (1 << j))[rank]
                    if acc in fresh:
                        fresh.discard(acc)
                        out.append("v_mul_f32 %s, %s, %s" % (acc, x, y))
                    elif sign > 0:
                        out.append("v_fmac_f32 %s, %s, %s" % (acc, x, y))
                    else:
                        out.append("v_fma_f32 %s, -%s, %s, %s" % (acc, x, y, acc))
    return out


def sum_handlers():
    """Transition sums of the qubit behind register bit j, from which the derivatives with respect to its angles follow:
    Im <lambda| P |psi> for the axes P that its unitary's rotations need.  B keeps one sum per lane for the S2 after the
    unitary; S1, S2 and S3 add one, two and three up over the wavefront and write a record of four floats: [A A A A],
    [A A B B] (A: its own axis, B: what was kept) and [X Z Y 0].
    A unitary of one rotation R needs its axis, which commutes with it; of two, R1 R0, the axis of R1 before the inverse
    unitary and that of R0 after it; of three, all axes after it.  So 4, 8 or 12 multiply-adds a pair beside the 8 to 20
    of the two unitaries; adding up over the lanes takes 12 to 14 instructions: v_permlane32_swap and
    v_permlane16_swap halve the lanes that hold a value by swapping it with another's (or its own copy's) half, four
    row rotations add up the rest.  s_nop 1: what these instructions need after their source was written."""
    H = []
    m = ["%%[m%d]" % k for k in range(4)]

    def swap(bits, a, b):
        return ["s_nop 1", "v_permlane%d_swap_b32 %s, %s" % (bits, a, b), "v_add_f32 %s, %s, %s" % (a, a, b)]

    rows = []
    for k in (8, 4, 2, 1):
        rows += ["s_nop 1", "v_add_f32_dpp %s, %s, %s row_ror:%d row_mask:0xf bank_mask:0xf" % (m[0], m[0], m[0], k)]
    write = rows + ["v_lshrrev_b32 %[t0], 4, %[thr]", "v_lshlrev_b32 %[t0], 2, %[t0]", "s_mov_b64 exec, s[74:75]",
                    "global_store_dword %[t0], " + m[0] + ", s[72:73]", "s_mov_b64 exec, -1",
                    "s_add_u32 s72, s72, %[sstep]", "s_addc_u32 s73, s73, 0"]
    twice = ["v_mov_b32 %s, %s" % (m[2], m[0])] + swap(16, m[0], m[2])      # both rows of a half from the row sums
    for j in range(R):
        for axis in AXES:
            H.append(("B%d%s" % (j, axis), NEXT_WORD + lane_sums(j, axis, ["%[kept]"]) + DISPATCH))
            own = lane_sums(j, axis, [m[0]])
            H.append(("S1%d%s" % (j, axis), NEXT_WORD + own + ["v_mov_b32 %s, %s" % (m[1], m[0])] + swap(32, m[0], m[1]) +
                      twice + write + DISPATCH))
            H.append(("S2%d%s" % (j, axis), NEXT_WORD + own + swap(32, m[0], "%[kept]") + twice + write + DISPATCH))
        H.append(("S3%d" % j, NEXT_WORD + lane_sums(j, AXES, m[:3]) + ["v_mov_b32 %s, 0" % m[3]] + swap(32, m[0], m[1]) +
                  swap(32, m[2], m[3]) + swap(16, m[0], m[2]) + write + DISPATCH))
    return H


def direct_handlers(pair=False):
    """[(name, lines)] in the order of the text; a line that ends in ':' is a local label."""
    H = []

    def states(lines):                           # what is done to psi, and the same to lambda
        return lines + of_lambda(lines) if pair else lines

    def flips(elems):
        return ["v_xor_b32 %%[%s%d], 0x80000000, %%[%s%d]" % (p, k, p, k) for k in elems for p in "ri"]

    # unitaries: the stub adds the register bit's part to the offset that the entry holds; _S looks for the
    # shifted matrix of a gradient row first
    for j in range(R):
        go = (["s_add_u32 s54, s54, %d" % (j * u_stride(pair))] if j else []) + [
            "s_add_u32 s64, s36, s54", "s_addc_u32 s65, s37, 0", "s_setpc_b64 s[64:65]"]
        H.append(("U%d" % j, go))
        if not pair:
            H.append(("US%d" % j, ["s_cmp_eq_u32 s43, %[ovrid]", "s_cbranch_scc1 L_dovr%d_%%=" % j] + go))
    for j in range(R):
        pairs = [(i, i | (1 << j)) for i in range(NR) if not i & (1 << j)]
        body = [ln for a, b in pairs for ln in u_pair(a, b)]
        if not pair:
            H.append(("G%d" % j, ["v_mov_b32 %%[m%d], s%d" % (k, 48 + k) for k in range(8)] + ["L_dgj%d_%%=:" % j] +
                      NEXT_ENTRY + NEXT_WORD + body + DISPATCH))
            H.append(("GS%d" % j, ["s_cmp_eq_u32 s43, %[ovrid]", "s_cbranch_scc0 L_dG%d_%%=" % j, "L_dovr%d_%%=:" % j,
                               "s_load_dwordx8 s[56:63], %[ovr], 0x0", "s_waitcnt lgkmcnt(0)"] +
                  ["v_mov_b32 %%[m%d], s%d" % (k, 56 + k) for k in range(8)] + ["s_branch L_dgj%d_%%=" % j]))
    # gradient rows that turn an angle by pi: the turn as a matrix before the unitary (UT), or by itself where the unitaries
    # are in the start state (V), in the row that names it
    if not pair:
        turn = lambda j: ["s_load_dwordx8 s[56:63], %[ovr], 0x0", "s_waitcnt lgkmcnt(0)"] + [
            "v_mov_b32 %%[m%d], s%d" % (k, 56 + k) for k in range(8)] + [
            ln for i in range(NR) if not i & (1 << j) for ln in u_pair(i, i | (1 << j))]
        for j in range(R):
            H.append(("UT%d" % j, ["s_cmp_eq_u32 s43, %[ovrid]", "s_cbranch_scc0 L_dU%d_%%=" % j] + turn(j) +
                      ["s_branch L_dU%d_%%=" % j]))
            H.append(("V%d" % j, ["s_mov_b32 s70, s43"] + NEXT_WORD +
                      ["s_cmp_eq_u32 s70, %[ovrid]", "s_cbranch_scc0 L_dV%dx_%%=" % j] + turn(j) +
                      ["L_dV%dx_%%=:" % j] + DISPATCH))
    # the scalar of a group by itself: 4 instructions an amplitude, as many as the whole matrix takes above the
    # cheapest form; it rounds all amplitudes alike, where a rounded matrix changes the lengths of its two columns by
    # different amounts, which shows in <Z> of the qubit in full (3e-8)
    scaled = []
    for k in range(NR):
        r, i = "%%[r%d]" % k, "%%[i%d]" % k
        scaled += ["v_mul_f32 %%[t0], %%[m1], %s" % i, "v_mul_f32 %%[t1], %%[m1], %s" % r,
                   "v_fma_f32 %s, %%[m0], %s, -%%[t0]" % (r, r), "v_fma_f32 %s, %%[m0], %s, %%[t1]" % (i, i)]
    H.append(("M", ["v_mov_b32 %[m0], s48", "v_mov_b32 %[m1], s49"] + NEXT_ENTRY + NEXT_WORD + states(scaled) + DISPATCH))
    # CNOTs: inside the register run, chains of them, control elsewhere (a mask of the lane's index bits: one
    # bit, or the parity of several), target behind a lane bit
    for jt in range(R):
        for jc in range(R):
            if jt != jc:
                H.append(("X%d%d" % (jt, jc), NEXT_WORD + states(move_pairs(
                    [(i, i | (1 << jt)) for i in range(NR) if (i >> jc) & 1 and not (i >> jt) & 1])) + DISPATCH))
    for k, chain in enumerate(CX_CHAINS):
        H.append(("C%d" % k, NEXT_WORD + states(chain_moves(*chain)) + DISPATCH))
    for j in range(R):
        swap = states(move_pairs([(i, i | (1 << j)) for i in range(NR) if not (i >> j) & 1]))
        for name, cond in (("D", []), ("P", ["v_bcnt_u32_b32 %[tc], %[tc], 0", "v_and_b32 %[tc], 1, %[tc]"])):
            done = "L_d%s%dx_%%=" % (name, j)
            H.append(("%s%d" % (name, j), ["v_and_b32 %[tc], s43, %[e0]"] + cond + NEXT_WORD +
                      ["v_cmp_ne_u32 vcc, 0, %[tc]", "s_and_saveexec_b64 s[68:69], vcc", "s_cbranch_execz " + done] +
                      swap + [done + ":", "s_mov_b64 exec, s[68:69]"] + DISPATCH))
    for j in range(R):
        high = [k for k in range(NR) if (k >> j) & 1]
        for b, perm in ((0, "[1,0,3,2]"), (1, "[2,3,0,1]")):
            H.append(("N%d%d" % (j, b), NEXT_WORD + states([
                "v_mov_b32_dpp %%[%s%d], %%[%s%d] quad_perm:%s row_mask:0xf bank_mask:0xf" % (p, k, p, k, perm)
                for k in high for p in "ri"]) + DISPATCH))
        H.append(("N%d" % j, ["v_xor_b32 %[tc], s43, %[thr]", "v_and_b32 %[tc], 63, %[tc]",
                              "v_lshlrev_b32 %[tc], 2, %[tc]"] + NEXT_WORD +
                  states(["ds_bpermute_b32 %%[%s%d], %%[tc], %%[%s%d]" % (p, k, p, k) for k in high for p in "ri"]) + DISPATCH))
    # CZ rungs: inside the run (any set of the three), one end in it, none
    for mask in range(1, 1 << CZ_RUNGS):
        H.append(("ZR%d" % mask, NEXT_WORD + states(flips(cz_elements(mask))) + DISPATCH))
    for j in range(R):
        H.append(("ZM%d" % j, ["v_and_b32 %[tc], s43, %[e0]"] + NEXT_WORD +
                  ["v_cmp_ne_u32 vcc, 0, %[tc]", "s_and_saveexec_b64 s[68:69], vcc", "s_cbranch_execz L_dZM%dx_%%=" % j] +
                  states(flips([k for k in range(NR) if (k >> j) & 1])) + ["L_dZM%dx_%%=:" % j, "s_mov_b64 exec, s[68:69]"] +
                  DISPATCH))
    H.append(("ZL", ["v_lshrrev_b32 %[tc], 1, %[e0]", "v_and_b32 %[tc], %[tc], %[e0]", "v_and_b32 %[tc], s43, %[tc]",
                     "v_bcnt_u32_b32 %[tc], %[tc], 0", "v_and_b32 %[tc], 1, %[tc]"] + NEXT_WORD +
              ["v_cmp_ne_u32 vcc, 0, %[tc]", "s_and_saveexec_b64 s[68:69], vcc", "s_cbranch_execz L_dZLx_%="] +
              states(flips(range(NR))) + ["L_dZLx_%=:", "s_mov_b64 exec, s[68:69]"] + DISPATCH))
    if pair:
        H += sum_handlers()
    H.append(("END", ["s_branch L_dexit_%="]))
    # transposes: W<s> writes the real parts in layout s and goes on to the target layout's R code (argument: its
    # offset / 64, bit 16: the exchange crosses wavefronts, bit 17: barrier before the writes); that reads
    # them and comes back to W<s>'s imaginary half, and so on, in the paired form with lambda's parts after psi's
    def cross(name):
        return ["s_bitcmp1_b32 s70, 16", "s_cbranch_scc0 " + name, "s_waitcnt lgkmcnt(0)", "s_barrier", name + ":"]

    def at(s, k):
        return 4 * padded(k << s)

    parts = PARTS if pair else PARTS[:2]
    delta = ["s_add_u32 s66, s66, %d" % X_DELTA, "s_addc_u32 s67, s67, 0"]
    back = ["s_add_u32 s64, s64, %d" % X_DELTA, "s_addc_u32 s65, s65, 0"]
    for nth, (sub, part) in enumerate(parts):
        for s in range(LAYOUTS):
            w = ["ds_write_b32 %%[ldsb], %%[%s%d] offset:%d" % (part, k, at(s, k)) for k in range(NR)]
            name = "W%s%d" % (sub, s)
            if nth == 0:
                H.append((name, ["s_mov_b32 s70, s43"] + NEXT_WORD +
                          ["s_bitcmp1_b32 s70, 17", "s_cbranch_scc0 L_dW%db_%%=" % s, "s_barrier", "L_dW%db_%%=:" % s] + w +
                          ["s_and_b32 s66, s70, 0xffff", "s_lshl_b32 s66, s66, 6", "s_add_u32 s66, s36, s66",
                           "s_addc_u32 s67, s37, 0", "s_add_u32 s64, s36, @WI%d" % s, "s_addc_u32 s65, s37, 0",
                           "s_setpc_b64 s[66:67]"]))
            else:
                H.append((name, cross("L_d%sb_%%=" % name) + w + delta + (back if nth + 1 < len(parts) else []) +
                          ["s_setpc_b64 s[66:67]"]))
    for nth, (sub, part) in enumerate(parts):
        for s in range(LAYOUTS):
            name = "R%s%d" % (sub, s)
            r = cross("L_d%sb_%%=" % name) + ["ds_read_b32 %%[%s%d], %%[ldsn] offset:%d" % (part, k, at(s, k)) for k in range(NR)]
            if nth == 0:
                r = lane_address(s) + r
            H.append((name, r + (["v_mov_b32 %[ldsb], %[ldsn]"] + DISPATCH if nth + 1 == len(parts) else ["s_setpc_b64 s[64:65]"])))
    if pair:
        H = [(name, [ln.replace("%[t2]", "%[m0]").replace("%[tc]", "%[m1]") for ln in lines]) for name, lines in H]
    return H


def lane_address(s):
    """The lane's part of its elements' LDS byte address in layout s, and its index e0."""
    out = ["v_lshrrev_b32 %%[t0], %d, %%[thr]" % s, "v_and_b32 %%[t1], %d, %%[thr]" % ((1 << s) - 1),
           "v_lshl_or_b32 %%[t0], %%[t0], %d, %%[t1]" % (s + R),             # tau of the lane's element 0
           "v_lshrrev_b32 %[t1], 5, %[t0]", "v_lshl_add_u32 %[t1], %[t1], 1, %[t0]",
           "v_lshlrev_b32 %[ldsn], 2, %[t1]"]
    return out + ["v_lshrrev_b32 %[t1], %[c], %[t0]", "v_and_b32 %[t2], %[cmask], %[t0]",
                  "v_lshlrev_b32 %[t1], %[w], %[t1]", "v_or_b32 %[t2], %[tb], %[t2]", "v_or_b32 %[e0], %[t1], %[t2]"]


def direct_layout(pair=False):
    """({name: byte offset}, first free offset): unitaries' sequences first, at fixed strides."""
    off, pos = {}, 64 * (3 if pair else 2)       # the block's own start takes two or three lines
    steps = 4 if pair else 2
    for form in FORMS:
        for core in range(len(CORES)):
            off["F%s%d" % (form, core)] = pos
            pos += u_stride(pair) * R
    group = {"W": 0, "R": 0}
    for name, lines in direct_handlers(pair):
        m = re.fullmatch(r"(W|R)(L?I?)(\d+)", name)
        if m:                                    # 256-byte places: W, WI, R, RI by layout, paired W, WI, WL, WLI, ...
            if not group["W"]:
                pos = (pos + 255) // 256 * 256
                group["W"], group["R"] = pos, pos + steps * X_DELTA
                pos += 2 * steps * X_DELTA
            off[name] = group[m.group(1)] + [sub for sub, _ in PARTS].index(m.group(2)) * X_DELTA + 256 * int(m.group(3))
            continue
        off[name] = pos
        pos += (sum(size_of(ln) for ln in lines if not ln.endswith(":")) + 63) // 64 * 64
    return off, pos


def gen_direct(pair=False):
    off, end = direct_layout(pair)
    L = [".p2align 6", "L_dbase_%=:",
         "s_getpc_b64 s[36:37]", "s_sub_u32 s36, s36, 4", "s_subb_u32 s37, s37, 0",
         "s_mov_b64 s[38:39], %[ops]", "s_mov_b64 s[44:45], %[mats]", "s_mov_b32 s40, 0", "s_mov_b32 s41, %[first]",
         "s_load_dwordx2 s[42:43], s[38:39], 0x0", "s_load_dwordx8 s[48:55], s[44:45], s41"]
    if pair:
        L += ["s_mov_b64 s[72:73], %[sums]", "s_mov_b32 s74, 0x10001", "s_mov_b32 s75, 0x10001"]
    L += DISPATCH
    bodies = []
    for form in FORMS:
        for core, name in enumerate(CORES):
            used = sorted({int(m) for ln in rot_pair(0, 1, form, name) for m in re.findall(r"%\[m(\d)\]", ln)})
            for j in range(R):
                body = []
                for i in range(NR):
                    if not i & (1 << j):
                        body += rot_pair(i, i | (1 << j), form, name)
                body = ["v_mov_b32 %%[m%d], s%d" % (k, 48 + k) for k in used] + NEXT_ENTRY + NEXT_WORD + body + (
                    of_lambda(body) if pair else [])
                bodies.append((off["F%s%d" % (form, core)] + j * u_stride(pair), "F%s%d%d" % (form, core, j), body + DISPATCH))
    for name, lines in direct_handlers(pair):
        bodies.append((off[name], name, [re.sub(r"@(\w+)", lambda m: str(off[m.group(1)]), ln) for ln in lines]))
    for pos, name, lines in sorted(bodies):
        L.append(".org L_dbase_%%=+%d, 0" % pos)
        L.append("L_d%s_%%=:" % name)
        L += lines
    L.append(".org L_dbase_%%=+%d, 0" % end)
    L.append("L_dexit_%=:")
    return L


def direct_constants(pair=False):
    """C++ constants the host needs to write operation words and the matrix builder to write entries."""
    off, _ = direct_layout(pair)
    rows = lambda names: ", ".join(str(off[n]) for n in names)
    j4 = range(R)
    c = [
        "namespace qsv { struct %s {" % ("paired" if pair else "direct"),
        "// byte offsets of the code of each operation in the block (see gen_direct in the generator)",
        "static constexpr unsigned kU[4] = {%s};" % rows("U%d" % j for j in j4),
        "static constexpr unsigned kG[4] = {%s}, kUShift[4] = {%s}, kGShift[4] = {%s};\n"
        "static constexpr unsigned kUTurn[4] = {%s}, kTurn[4] = {%s};" % tuple(
            rows("%s%d" % (name, j) for j in j4) for name in ("G", "US", "GS", "UT", "V")) if not pair else
        "static constexpr unsigned kBefore[4][3] = {%s}, kSum1[4][3] = {%s}, kSum2[4][3] = {%s}, kSum3[4] = {%s};" % (
            *(", ".join("{%s}" % rows("%s%d%s" % (k, j, x) for x in AXES) for j in j4) for k in ("B", "S1", "S2")),
            rows("S3%d" % j for j in j4)),
        "static constexpr unsigned kCx[4][4] = {%s};   // [target][control]" % ", ".join(
            "{%s}" % ", ".join(str(off.get("X%d%d" % (t, c), 0)) for c in j4) for t in j4),
        "static constexpr unsigned kChain[%d] = {%s};" % (len(CX_CHAINS), rows("C%d" % k for k in range(len(CX_CHAINS)))),
        "static constexpr unsigned kCxBit[4] = {%s}, kCxParity[4] = {%s};" % (rows("D%d" % j for j in j4), rows("P%d" % j for j in j4)),
        "static constexpr unsigned kCxQuad[4][2] = {%s}, kCxLane[4] = {%s};" % (
            ", ".join("{%s}" % rows("N%d%d" % (j, b) for b in (0, 1)) for j in j4), rows("N%d" % j for j in j4)),
        "static constexpr unsigned kCz[8] = {0, %s}, kCzMix[4] = {%s}, kCzLane = %d, kScale = %d, kEnd = %d;" % (
            rows("ZR%d" % m for m in range(1, 8)), rows("ZM%d" % j for j in j4), off["ZL"], off["M"], off["END"]),
        "static constexpr unsigned kWrite[%d] = {%s};" % (LAYOUTS, rows("W%d" % s for s in range(LAYOUTS))),
        "static constexpr unsigned kRead[%d] = {%s};" % (LAYOUTS, rows("R%d" % s for s in range(LAYOUTS))),
        "static constexpr unsigned kSeq0 = %d, kSeqStride = %d;   // code of a factored unitary: kSeq0 + sequence * kSeqStride" % (
            off["Fnone0"], u_stride(pair) * R),
        "}; }",
    ]
    return c


def render():
    out = ["// Generated by gen_gate_asm.py -- do not edit by hand.",
           "// Inline-assembly gate interpreter of the fused pass kernel; see the generator for the",
           "// register map and the reason it is assembly.  _2P: transposes through two LDS planes",
           "// (real, imaginary) at once; _1P: through one plane, real parts first.  _ROWS: for tiles that",
           "// hold several state rows (returns at a unitary whose matrix depends on the row).",
           "#pragma once"]
    for planes in (2, 1):
        for perlane in (False, True):
            out.append("#define QSV_GATE_LOOP_ASM_%dP%s \\" % (planes, "_ROWS" if perlane else ""))
            for ln in gen(planes, perlane):
                out.append('    "%s\\n\\t" \\' % ln)
            out.append('    ""')
    for pair, name, last in ((False, "DIRECT", DIRECT_LAST), (True, "PAIRED", PAIR_LAST)):
        out.append("#define QSV_GATE_%s_ASM \\" % name)
        for ln in gen_direct(pair):
            out.append('    "%s\\n\\t" \\' % ln)
        out.append('    ""')
        regs = ", ".join('"s%d"' % i for i in range(DIRECT_FIRST, last + 1))
        out.append("#define QSV_GATE_%s_CLOBBERS %s, \"vcc\", \"scc\", \"memory\"" % (name, regs))
        out += direct_constants(pair)
    regs = ", ".join('"s%d"' % i for i in range(FIRST_SGPR, LAST_SGPR + 1))
    out.append("#define QSV_GATE_LOOP_CLOBBERS %s, \"vcc\", \"scc\", \"memory\"" % regs)
    return "\n".join(out) + "\n"


def write(path=None):
    path = path or os.path.join(os.path.dirname(os.path.abspath(__file__)), "qsv_gate_asm.h")
    text = render()
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)
    return path


if __name__ == "__main__":
    print(write())
