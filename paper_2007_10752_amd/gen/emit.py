"""Write the generated C++ headers under csrc/generated from the Appendix A
tables (des_tables.py) and the verified S-box networks (sbox_networks.txt).

    python -m paper_2007_10752_amd.gen.emit

Outputs
  des_tables_gen.h   PC-1 / PC-2 / rotation tables for the host key schedule
  bitslice_gen.h     bitsliced kernel: IP and FP as plane renaming, one
                     Feistel round (E and P as renaming, S-boxes as gates)
  bitslice_boxes_gen.h  the S-boxes one by one, for the split bitsliced kernel
  bitslice_keys_gen.h  host tables for the bitsliced kernel's key masks
  spbox_gen.h        table kernel: the 8 combined S-box+P tables and IP/FP as
                     delta swaps on a block held in two 32-bit words

Bit conventions used throughout the library: DES bit n (1..64) is bit
(7 - (n-1) % 8) of byte (n-1) // 8 (bit 1 = most significant bit of byte 0).
A block is read as two little-endian 32-bit words h = 0, 1 (bytes 0-3, 4-7),
so DES bit n sits in word (n-1)//32 at bit position 8*((n-1)//8 % 4) + 7 - (n-1)%8.
"""
import os

from . import des_tables as T
from .networks import (MASK_BASE, fold_network, format_networks, load_networks, second_use_plan,
                       verify_folded, verify_network)

HERE = os.path.dirname(os.path.abspath(__file__))
OUT_DIR = os.path.join(os.path.dirname(HERE), "csrc", "generated")

BANNER = ("// Generated by paper_2007_10752_amd/gen/emit.py from the DES tables of the\n"
          "// paper's Appendix A and the verified S-box networks.  Do not edit.\n")


def word_pos(n):
    """(word, bit position) of DES bit n (1..64) in the little-endian pair."""
    i, j = (n - 1) // 8, (n - 1) % 8
    return i // 4, (i % 4) * 8 + (7 - j)


def c_array(decl, vals, per_line=16):
    """``decl`` is the declaration up to the name, e.g. "static const int X"."""
    lines = []
    for i in range(0, len(vals), per_line):
        lines.append("    " + ", ".join(str(v) for v in vals[i:i + per_line]) + ",")
    return "%s[%d] = {\n%s\n};\n" % (decl, len(vals), "\n".join(lines))


# ---------------------------------------------------------------- key tables --

def emit_tables():
    s = [BANNER, "#pragma once\n#include <stdint.h>\n\n"]
    s.append("// Appendix A: permuted choice 1 (64 -> 56), 1-based source bits\n")
    s.append(c_array("static constexpr uint8_t kPC1", list(T.PC1), 14))
    s.append("// Appendix A: permuted choice 2 (56 -> 48), 1-based source bits\n")
    s.append(c_array("static constexpr uint8_t kPC2", list(T.PC2), 12))
    s.append("// Appendix A: left rotations of each 28-bit half, rounds 1..16\n")
    s.append(c_array("static constexpr uint8_t kShifts", list(T.SHIFTS), 16))
    return "".join(s)


def emit_replica_tables():
    """The Appendix A arrays the one-thread-per-bit comparison kernel reads
    at run time (1-based source positions; S-boxes box-major, then row,
    then column)."""
    s = [BANNER, "#pragma once\n#include <stdint.h>\n\n"]
    s.append("// Appendix A: initial permutation, 1-based source bits\n")
    s.append(c_array("static constexpr uint8_t kRepIP", list(T.IP), 16))
    s.append("// Appendix A: expansion of the right half, 1-based source bits\n")
    s.append(c_array("static constexpr uint8_t kRepE", list(T.E), 16))
    s.append("// Appendix A: S-boxes, value of box b, row r, column c at 64 b + 16 r + c\n")
    s.append(c_array("static constexpr uint8_t kRepS", [v for box in T.SBOX for row in box for v in row], 16))
    s.append("// Appendix A: straight permutation, 1-based source bits\n")
    s.append(c_array("static constexpr uint8_t kRepP", list(T.P), 16))
    s.append("// Appendix A: final permutation, 1-based source bits\n")
    s.append(c_array("static constexpr uint8_t kRepFP", list(T.FP), 16))
    return "".join(s)


# ------------------------------------------------------------ bitsliced ----

def plane_of(n):
    """Plane register of DES bit n after the in-lane 32x32 transposes:
    plane h*32 + p holds bit position p of word h of 32 blocks."""
    h, p = word_pos(n)
    return 32 * h + p


_PLANS = {}


def plan(nets=None):
    """second_use_plan of the networks (by default the committed ones),
    computed once per set of networks."""
    if nets is None:
        nets = load_networks()
    key = format_networks(nets)
    if key not in _PLANS:
        _PLANS[key] = second_use_plan(nets)
    return _PLANS[key]


def e_structure(nets=None):
    """How the expansion E feeds the S-boxes: E position e (0..47) reads
    right-half word E[e]-1.  16 words feed two positions: one is the word's
    primary use (its word carries that position's key mask), the other its
    second use (XORed with its own mask, or the mask folded into the gates),
    as second_use_plan chose for the networks."""
    second, _ = plan(nets)
    src = [T.E[e] - 1 for e in range(48)]
    primary, dup_of_e, dup_e = [None] * 32, [-1] * 48, []
    for e in range(48):
        if e in second:
            dup_of_e[e] = len(dup_e)
            dup_e.append(e)
        else:
            assert primary[src[e]] is None
            primary[src[e]] = e
    assert len(dup_e) == 16 and None not in primary
    return src, primary, dup_of_e, dup_e


def box_network(nets, box):
    """S-box `box`'s network as the kernels run it: with the masks of its
    folded second uses taken by the gates (fold_network), else as searched."""
    _, folded = plan(nets)
    fq = sorted(e % 6 for e in folded if e // 6 == box)
    return fold_network(nets[box], fq) if fq else dict(nets[box], folded=[])


def box_signals(box, src, dup_of_e, fnet, mask_of):
    """Declarations of a box's inputs and the signal names its gates use:
    x<q> is the right-half word (XORed with its second-use mask unless that
    mask is folded), the folded masks appear as mask_of(i), i the input's
    index among the box's second uses."""
    decl, names, di = [], {}, 0
    for q in range(6):
        e = 6 * box + q
        if dup_of_e[e] < 0:
            decl.append("        const uint32_t x%d = r[%d];\n" % (q, src[e]))
        elif q in fnet["folded"]:
            decl.append("        const uint32_t x%d = r[%d];  // mask folded into its gates\n"
                        % (q, src[e]))
            names[MASK_BASE + q] = mask_of(di, dup_of_e[e])
            di += 1
        else:
            decl.append("        const uint32_t x%d = r[%d] ^ %s;\n" % (q, src[e], mask_of(di, dup_of_e[e])))
            di += 1
        names[q] = "x%d" % q
    return decl, names


def out_word():
    """Half-word that S-box output (box, q) is XORed into (straight
    permutation P as renaming), indexed 4*box + q."""
    pinv = {T.P[j] - 1: j for j in range(32)}
    return [pinv[m] for m in range(32)]


# Layout of a direction's key masks (0 or ~0 words) as one table (the kernels widen
# a round's at a time): round t (0..47) takes 64 words at 64*t, 8 per S-box:
# box j at 64*t + 8*j holds [0..3] the masks folded into the XORs of its
# outputs q = 0..3 into the other half, [4..7] the masks of its second-use
# expansion inputs in input order (box_dups(j); unused slots 0); then 32
# words each of: the initial mask of R (Y), the re-masks of X before round 16
# and of Y before round 32, and the final unmask of X.
BS_BOX_MASKS = 8
BS_ROUND_MASKS = 8 * BS_BOX_MASKS
BS_INIT_Y = 48 * BS_ROUND_MASKS
BS_REMASK_16 = BS_INIT_Y + 32
BS_REMASK_32 = BS_REMASK_16 + 32
BS_FINAL_X = BS_REMASK_32 + 32
BS_NMASK = BS_FINAL_X + 32


def box_dups(box):
    """Second-use indices k (0..15) of S-box `box`'s inputs, in input order."""
    _, _, dup_of_e, _ = e_structure()
    return [dup_of_e[6 * box + q] for q in range(6) if dup_of_e[6 * box + q] >= 0]


def emit_bitslice(nets):
    ip_l = [plane_of(T.IP[i]) for i in range(32)]
    ip_r = [plane_of(T.IP[32 + i]) for i in range(32)]
    # output plane q carries DES bit n with plane_of(n) == q; its value is
    # preoutput bit FP[n-1], preoutput = R16 || L16
    fp_src = [0] * 64
    for n in range(1, 65):
        fp_src[plane_of(n)] = T.FP[n - 1] - 1  # 0..31 -> R16[i], 32..63 -> L16[i-32]

    s = [BANNER, "#pragma once\n#include <stdint.h>\n\n"]
    s.append("// Initial permutation as renaming: L[i] / R[i] read plane BS_IP_L[i] / BS_IP_R[i]\n")
    s.append(c_array("static constexpr int BS_IP_L", ip_l))
    s.append(c_array("static constexpr int BS_IP_R", ip_r))
    s.append("// Final permutation as renaming: output plane q is preoutput bit BS_FP_SRC[q]\n"
             "// (preoutput = R16 || L16: 0..31 from R16, 32..63 from L16)\n")
    s.append(c_array("static constexpr int BS_FP_SRC", fp_src))
    total = sum(len(n["gates"]) for n in nets.values())
    _, folded = plan(nets)
    s.append("\n// S-box gate counts: %s (total %d per round)\n" % (
        ", ".join("S%d=%d" % (b + 1, len(nets[b]["gates"])) for b in range(8)), total))
    s.append("#define BS_SBOX_GATES_PER_ROUND %d\n" % total)
    s.append("// XORs per round: 32 of S-box outputs into the other half, and the second\n"
             "// uses whose masks are not folded into the gates (%d of 16 are)\n" % len(folded))
    s.append("#define BS_XORS_PER_ROUND %d\n\n" % (32 + 16 - len(folded)))
    s.append(emit_round_piped(nets))
    return "".join(s)


def emit_round_piped(nets):
    """One Feistel round with the key masks of each S-box in registers, made D
    boxes before they are used."""
    src, primary, dup_of_e, dup_e = e_structure(nets)
    ow = out_word()
    s = ["\n// Number of second-use inputs of each S-box (mask words e[] it reads).\n",
         c_array("static constexpr int BS_BOX_NDUP", [len(box_dups(b)) for b in range(8)]),
         "\n// Key masks of one S-box in registers: o[q] is folded into the XOR of output q\n"
         "// into the other half, e[i] is the mask of the box's i-th second-use input.\n"
         "struct BsBoxMasks {\n    uint32_t o[4], e[4];\n};\n\n"
         "// One Feistel round on 32 blocks per lane (Sec. III-B): d ^= P(S(E(r) ^ K)).\n"
         "// The halves are stored XORed with key masks: each word of r already carries the\n"
         "// round-key bit of its primary expansion position, so only second uses need their\n"
         "// mask: XORed in, or taken as the third operand of the gates that read the input;\n"
         "// the output masks re-mask the updated words of d for their next use.  Masks are\n"
         "// laid out by round and S-box (8 words per box, 64 per round: o[0..3], e[0..3])\n"
         "// and software-pipelined D boxes ahead: before box j\n"
         "// runs, load(pm[(j + D) % 8], q, n) requests the masks of the box D places\n"
         "// later, q = p + 8 * (j + D), or past the last box pn + 8 * (j + D - 8) (pn: the\n"
         "// next round's masks).\n"
         "// A scheduling barrier between boxes keeps each request and each box's\n"
         "// arithmetic in place, so the request's latency overlaps D boxes of work.\n"
         "// On entry pm[0..D-1] hold this round's first D boxes; on exit the next round's.\n"
         "// n = BS_BOX_NDUP of the requested box: load fills o[0..3] and e[0..n-1] only.\n"
         "// P: the pointer type of p and pn (a generic or an LDS pointer).\n"
         "template <int D, class LOAD, class P>\n"
         "__device__ __forceinline__ void bs_round_piped(uint32_t (&d)[32], const uint32_t (&r)[32],\n"
         "                                               P p, P pn, BsBoxMasks (&pm)[8],\n"
         "                                               const LOAD &load) {\n"
         "    static_assert(D >= 1 && D <= 7, \"pipeline depth\");\n"]
    for box in range(8):
        net = box_network(nets, box)
        s.append("    {  // S%d\n" % (box + 1))
        s.append("        __builtin_amdgcn_sched_barrier(0);\n")
        s.append("        load(pm[(%d + D) %% 8],\n"
                 "             %d + D < 8 ? p + %d * (%d + D) : pn + %d * (%d + D - 8),\n"
                 "             BS_BOX_NDUP[(%d + D) %% 8]);\n"
                 % (box, box, BS_BOX_MASKS, box, BS_BOX_MASKS, box, box))
        s.append("        const BsBoxMasks &m = pm[%d];\n" % box)
        decl, names = box_signals(box, src, dup_of_e, net, lambda i, k: "m.e[%d]" % i)
        s.extend(decl)
        for i, (a, b, c, imm) in enumerate(net["gates"]):
            nm = "g%d" % (6 + i)
            s.append("        const uint32_t %s = __builtin_amdgcn_bitop3_b32(%s, %s, %s, 0x%02x);\n"
                     % (nm, names[a], names[b], names[c], imm))
            names[6 + i] = nm
        for q, (sig, neg) in enumerate(net["outs"]):
            j = ow[4 * box + q]
            s.append("        d[%d] = __builtin_amdgcn_bitop3_b32(d[%d], %s, m.o[%d], 0x%02x);\n"
                     % (j, j, names[sig], q, 0x69 if neg else 0x96))
        s.append("    }\n")
    s.append("}\n")
    return "".join(s)


def emit_bitslice_boxes(nets):
    """The S-boxes as separate functions, for kernels in which a wave runs
    some of them only: bs_box<J>(x, d, m) reads the box's six right-half
    words x (raw, in input order), XORs its outputs and their re-masks
    m.o[q] into the four words d[q] of the other half that they land in, and
    takes the second-use masks m.e[i] as bs_round_piped does."""
    _, _, dup_of_e, _ = e_structure(nets)
    s = [BANNER, "#pragma once\n#include <stdint.h>\n\n#include \"bitslice_gen.h\"\n\n",
         "// One S-box on 32 blocks per lane: d[q] ^= output q ^ m.o[q], x the box's six\n"
         "// inputs as right-half words, m.e[i] the mask of its i-th second-use input.\n"
         "template <int J>\n"
         "__device__ __forceinline__ void bs_box(const uint32_t *x, uint32_t *d, const BsBoxMasks &m);\n"]
    for box in range(8):
        net = box_network(nets, box)
        s.append("\ntemplate <>\n__device__ __forceinline__ void bs_box<%d>(const uint32_t *x, uint32_t *d,\n"
                 "                                           const BsBoxMasks &m) {  // S%d\n" % (box, box + 1))
        names, di = {}, 0
        for q in range(6):
            names[q] = "x%d" % q
            masked = dup_of_e[6 * box + q] >= 0
            if masked and q in net["folded"]:
                names[MASK_BASE + q] = "m.e[%d]" % di
            s.append("    const uint32_t x%d = x[%d]%s;\n"
                     % (q, q, " ^ m.e[%d]" % di if masked and q not in net["folded"] else ""))
            di += masked
        for i, (a, b, c, imm) in enumerate(net["gates"]):
            nm = "g%d" % (6 + i)
            s.append("    const uint32_t %s = __builtin_amdgcn_bitop3_b32(%s, %s, %s, 0x%02x);\n"
                     % (nm, names[a], names[b], names[c], imm))
            names[6 + i] = nm
        for q, (sig, neg) in enumerate(net["outs"]):
            s.append("    d[%d] = __builtin_amdgcn_bitop3_b32(d[%d], %s, m.o[%d], 0x%02x);\n"
                     % (q, q, names[sig], q, 0x69 if neg else 0x96))
        s.append("}\n")
    return "".join(s)


def emit_bitslice_keys():
    """Host-side tables for building the bitsliced kernel's key masks."""
    src, primary, dup_of_e, dup_e = e_structure()
    s = [BANNER, "#pragma once\n#include <stdint.h>\n\n"]
    s.append("// Expansion E (Appendix A): source word of each of the 48 S-box inputs,\n"
             "// the primary input of each word, and the 16 second-use inputs in order.\n")
    s.append(c_array("static constexpr int kBsESrc", src))
    s.append(c_array("static constexpr int kBsPrimaryE", primary))
    s.append(c_array("static constexpr int kBsDupE", dup_e))
    s.append("// Straight permutation P: half-word receiving S-box output 4*box+q.\n")
    s.append(c_array("static constexpr int kBsOutWord", out_word()))
    bd = []
    for box in range(8):
        ks = box_dups(box)
        assert len(ks) <= 4
        bd += ks + [-1] * (4 - len(ks))
    s.append("// Second-use index k of mask slot 4 + i of S-box j: kBsBoxDup[4*j + i] (-1: unused).\n")
    s.append(c_array("static constexpr int kBsBoxDup", bd))
    s.append("\n// Places of the masks widened from the key words, as a table: round t, box j at\n"
             "// kBsRoundMasks*t + kBsBoxMasks*j (outputs 0..3, then second uses); then the four\n"
             "// 32-word extra groups.  The kernels use a box's kBsBoxMasks places (a row of the\n"
             "// batched kernel's table), the CPU emulation of the tests the whole.\n")
    s.append("enum { kBsBoxMasks = %d, kBsRoundMasks = %d, kBsInitY = %d, kBsRemask16 = %d,\n"
             "       kBsRemask32 = %d, kBsFinalX = %d, kBsNumMasks = %d };\n"
             % (BS_BOX_MASKS, BS_ROUND_MASKS, BS_INIT_Y, BS_REMASK_16, BS_REMASK_32, BS_FINAL_X,
                BS_NMASK))
    return "".join(s)


# ------------------------------------------------------------ table kernel --

def sp_tables():
    """SP[s][v]: the 32-bit f contribution of S-box s on 6-bit input v, with
    f bit j (1..32) at bit position 32 - j."""
    pinv = {T.P[j] - 1: j for j in range(32)}
    out = []
    for box in range(8):
        for v in range(64):
            row = ((v >> 5) << 1) | (v & 1)
            col = (v >> 1) & 0xF
            val = T.SBOX[box][row][col]
            w = 0
            for q in range(4):
                if (val >> (3 - q)) & 1:
                    j = pinv[4 * box + q] + 1
                    w |= 1 << (32 - j)
            out.append(w)
    return out


# IP and FP for the table kernel.  Both are bit-permute-complement (BPC)
# permutations: with the block held big-endian in a 64-bit register (DES bit
# n at register bit e = 64 - n), the destination index of every bit is its
# source index with the six index bits permuted and some of them
# complemented.  Such a permutation is a product of exchanges of two index
# bits (optionally complementing both) and complements of one index bit;
# each is one delta swap on the register.  The register is two 32-bit
# words, hi (index bit 5 = 1) and lo.


def bpc_form(dest):
    """dest[e] = destination register index of source index e (0..63).
    Returns (sigma, comp) with bit k of dest[e] == bit sigma[k] of e XOR
    comp[k] for all e, or raises if dest is not BPC."""
    sigma, comp = [], []
    for k in range(6):
        found = None
        for src in range(6):
            for c in (0, 1):
                if all(((dest[e] >> k) & 1) == (((e >> src) & 1) ^ c) for e in range(64)):
                    found = (src, c)
        if found is None:
            raise ValueError("not a bit-permute-complement permutation")
        sigma.append(found[0])
        comp.append(found[1])
    return sigma, comp


def bpc_steps(sigma, comp):
    """Index-bit exchanges and complements taking the identity to (sigma,
    comp): a list of ("x", a, b, complement_both) and ("c", a)."""
    pos = [[k, 0] for k in range(6)]  # index bit k now holds source bit pos[k][0] ^ pos[k][1]
    steps = []
    for k in range(5, -1, -1):
        j = next(i for i in range(6) if pos[i][0] == sigma[k])
        if j != k:
            cboth = int(pos[j][1] != comp[k])
            pos[k], pos[j] = [pos[j][0], pos[j][1] ^ cboth], [pos[k][0], pos[k][1] ^ cboth]
            steps.append(("x", max(k, j), min(k, j), cboth))
    for k in range(6):
        if pos[k][1] != comp[k]:
            pos[k][1] ^= 1
            steps.append(("c", k))
    assert all(pos[k] == [sigma[k], comp[k]] for k in range(6))
    return steps


def _mask(pred):
    return sum(1 << e for e in range(32) if pred(e))


def bpc_code(steps):
    """C statements applying the steps to words hi, lo (uint32_t; t is a
    scratch word), and a Python function doing the same (for checking);
    returns (lines, n_ops, fn)."""
    lines, ops, prog = [], 0, []
    for st in steps:
        if st[0] == "x":
            _, a, b, cb = st
            if a < 5:
                d = (1 << a) + (1 << b) if cb else (1 << a) - (1 << b)
                m = _mask(lambda e: not (e >> a) & 1 and ((e >> b) & 1) == (0 if cb else 1))
                for w in ("hi", "lo"):
                    lines.append("    t = ((%s >> %d) ^ %s) & 0x%08xu; %s ^= t ^ (t << %d);"
                                 % (w, d, w, m, w, d))
                ops += 8
                prog.append(("in", d, m))
            else:
                sh = 1 << b
                m = _mask(lambda e: ((e >> b) & 1) == (0 if cb else 1))
                if cb:  # (0,0) <-> (1,1): lo position e pairs with hi position e + 2^b
                    lines.append("    t = ((hi >> %d) ^ lo) & 0x%08xu; lo ^= t; hi ^= t << %d;"
                                 % (sh, m, sh))
                    prog.append(("xc", sh, m))
                else:  # (0,1) <-> (1,0): lo position e pairs with hi position e - 2^b
                    lines.append("    t = ((hi << %d) ^ lo) & 0x%08xu; lo ^= t; hi ^= t >> %d;"
                                 % (sh, m, sh))
                    prog.append(("xp", sh, m))
                ops += 4
        else:
            a = st[1]
            if a == 5:
                lines.append("    t = hi; hi = lo; lo = t;")
                prog.append(("swap",))
            else:
                d = 1 << a
                m = _mask(lambda e: not (e >> a) & 1)
                for w in ("hi", "lo"):
                    lines.append("    %s = ((%s >> %d) & 0x%08xu) | ((%s & 0x%08xu) << %d);"
                                 % (w, w, d, m, w, m, d))
                ops += 6
                prog.append(("cm", d, m))

    def fn(hi, lo):
        M = 0xFFFFFFFF
        for op in prog:
            if op[0] == "in":
                _, d, m = op
                t = ((hi >> d) ^ hi) & m
                hi ^= t ^ ((t << d) & M)
                t = ((lo >> d) ^ lo) & m
                lo ^= t ^ ((t << d) & M)
            elif op[0] == "xc":
                _, sh, m = op
                t = ((hi >> sh) ^ lo) & m
                lo ^= t
                hi ^= (t << sh) & M
            elif op[0] == "xp":
                _, sh, m = op
                t = (((hi << sh) & M) ^ lo) & m
                lo ^= t
                hi ^= t >> sh
            elif op[0] == "swap":
                hi, lo = lo, hi
            else:
                _, d, m = op
                hi = ((hi >> d) & m) | ((hi & m) << d) & M
                lo = ((lo >> d) & m) | ((lo & m) << d) & M
        return hi, lo
    return lines, ops, fn


def bpc_of_table(table):
    """dest[] of a DES permutation table (output bit i+1 = input bit
    table[i]), in register indices (DES bit n at e = 64 - n)."""
    dest = [0] * 64
    for i, src in enumerate(table):
        dest[64 - src] = 64 - (i + 1)
    return dest


def check_bpc(fn, table):
    """fn on (hi, lo) must move every single bit as the table says."""
    for n in range(1, 65):
        e = 64 - n
        hi, lo = (1 << (e - 32), 0) if e >= 32 else (0, 1 << e)
        hi, lo = fn(hi, lo)
        got = (hi << 32) | lo
        want = 1 << (64 - (table.index(n) + 1))
        assert got == want, (n, hex(got), hex(want))


def emit_spbox():
    s = [BANNER, "#pragma once\n#include <stdint.h>\n\n"]
    s.append("// Combined S-box + straight permutation tables: SP[s*64 + v] is P applied to\n"
             "// the output of S-box s+1 on chunk v, f bit j at bit position 32 - j.\n")
    s.append(c_array("static __device__ const uint32_t SP_TABLE", ["0x%08xu" % v for v in sp_tables()], 8))
    sp = sp_tables()
    s.append("// The same by chunk: SP_BY_CHUNK[8 v + s].\n")
    s.append(c_array("static __device__ const uint32_t SP_BY_CHUNK",
                     ["0x%08xu" % sp[64 * box + v] for v in range(64) for box in range(8)], 8))
    for name, table, head, tail, what in (
            ("SP_IP(w0, w1, L, R)", T.IP,
             "    uint32_t hi = __builtin_bswap32(w0), lo = __builtin_bswap32(w1), t;",
             "    L = hi; R = lo;",
             "Initial permutation: (w0, w1) little-endian words of a block -> L, R\n"
             "// (bit i of a half at position 32 - i)"),
            ("SP_FP(Lf, Rf, o0, o1)", T.FP,
             "    uint32_t hi = Rf, lo = Lf, t;",
             "    o0 = __builtin_bswap32(hi); o1 = __builtin_bswap32(lo);",
             "Final permutation of preoutput Rf || Lf -> little-endian words o0, o1")):
        steps = bpc_steps(*bpc_form(bpc_of_table(table)))
        lines, ops, fn = bpc_code(steps)
        check_bpc(fn, list(table))
        s.append("\n// %s,\n// as %d delta swaps on the block held big-endian in two words\n"
                 "// (%d operations)\n" % (what, len(steps), ops + 2))
        s.append("#define %s do { \\\n" % name)
        s.extend(l + " \\\n" for l in [head] + lines + [tail])
        s.append("} while (0)\n")
    return "".join(s)


def main():
    nets = load_networks()
    for box in range(8):
        verify_network(box, nets[box])
        verify_folded(box, box_network(nets, box))
    os.makedirs(OUT_DIR, exist_ok=True)
    for name, text in (("des_tables_gen.h", emit_tables()),
                       ("bitslice_gen.h", emit_bitslice(nets)),
                       ("bitslice_boxes_gen.h", emit_bitslice_boxes(nets)),
                       ("bitslice_keys_gen.h", emit_bitslice_keys()),
                       ("spbox_gen.h", emit_spbox()),
                       ("replica_tables_gen.h", emit_replica_tables())):
        path = os.path.join(OUT_DIR, name)
        with open(path, "w") as f:
            f.write(text)
        print("wrote", path)


if __name__ == "__main__":
    main()
