#!/usr/bin/env python3
"""Writes mttkrp_pipe.inc: the software-pipelined inner loops of the streaming
kernel as inline assembly, one per instantiation (data type, row blocks RB,
column blocks JB) and load flavour (non-temporal or not, fp64 only).

Why assembly: the compiler places its waits for outstanding loads conservatively
around control flow, which keeps a wavefront from overlapping its own loads with
its own MFMAs.  The generated loop keeps D steps of loads in flight while the
MFMAs of an earlier step run.

One step = four tensor columns: the X loads of the tile's RB row blocks, the
loads of the inner factor's entries for the JB column blocks (both in the lane
layout the kernel defines: `Lay` / `LayRows` in mttkrp.hip), JB multiplies by
the sweep weight and RB * JB 16x16x4 MFMAs.  A run covers any n >= D consecutive
unmasked steps of one sweep: the X pointer and the factor offsets advance by
constant strides.  Both bases lie in scalar registers and are advanced by the
scalar unit; a lane's offsets from them are 32-bit registers that never change
(but see lane_pointers).
That matters in fp64: while an fp64 MFMA runs, the SIMD issues no vector
instruction, and a group of them between two MFMAs costs about 10 cycles and 2 to
4 more for each (register-only loop of RB = 2, JB = 4 steps: 568 cycles a step
with a 64-bit and two 32-bit pointer additions, 544 without, of 512 for the MFMAs
alone).  Operand sets live in a ring of S = D + 1 register sets at
fixed registers at the top of the wavefront's register budget (declared as
clobbers); the loads of step t go to set t mod S; every wait names how many
younger loads may still be outstanding (loads return in issue order).

Structure of a run: D steps are issued up front; then every pass through a ring
position checks whether steps are left, issues one more and consumes the oldest;
when none are left, the D steps in flight are consumed with waits that shrink
to 0 (one copy of that tail per ring position, because the registers differ).

Per instantiation the script picks the register budget (128 / 168 / 256
registers = 4 / 3 / 2 wavefronts per SIMD) and the depth D: the most
wavefronts for which accumulators + ring + an allowance for everything else the
kernel keeps live still fit, with 3 <= D <= 5.

Run by build.py before hipcc on every build; the output is a build product and is
not kept under version control.
"""
import os

D_MAX = 5
D_MIN = 3
S0 = 84                      # scalar registers of a run: X base, X step, base of the inner factor (two each)
XB, BB = "s[%d:%d]" % (S0, S0 + 1), "s[%d:%d]" % (S0 + 4, S0 + 5)
OTHERS = {2: 60, 1: 56}      # registers the rest of the kernel keeps live across a run (fp64, fp32)


def others(i):
    """The same for one instantiation.  (With twelve fp64 accumulators 60 would let D = 5 fit.  D = 4 takes sweeps of four
    steps through the run too, 124387 x 4^5 at R = 397, first mode 2.87 -> 2.16 ms, and is 1 % faster in the mean of 20 other
    calls.  The tile of three row and four column blocks reloads its lanes' offsets of X from scratch memory before each run
    either way; forming them from the lane number there instead gave nothing, 0.997 in the mean of 21 calls.)"""
    return OTHERS[i.w] + (14 if i.w == 2 and i.rb * i.jb == 12 else 0)


# A step's factor entries take the sweep's weight before they meet X, as everywhere else in the kernel.  Runs that summed X times
# the inner factor and multiplied the sums by the weight afterwards were 1 % faster in the mean (RB * JB * 4 FMAs a run for JB
# multiplies a step, 401 x 201 x 12 x 501 at R = 1000 2.5 %), but such a sum can leave the type's range where the weight brings
# it back (fp32: X 1e25, inner factor 1e15, outer 1e-15 became infinite), and a guard against that costs what they gain.  (fp32
# tiles of three or four row and four column blocks run three wavefronts a SIMD, though that keeps up to 66 registers in scratch
# memory outside the runs: two wavefronts without any took 1.02 times as long in the mean of 20 calls at R = 50 to 200, 16384 x 256
# x 64 at R = 128 508 -> 561 us.)


def lane_pointers(i):
    """Whether a run keeps X's addresses in 64-bit pointers of the lanes and advances them, and the inner factor's offsets, by
    vector additions, as the batches do.  Where a step has one or two MFMAs, or fp32 MFMAs for one column block, the scalar
    bases save little: their set-up per run and four dependent scalar additions a step cost as much, and wavefronts drift apart on
    short columns (fp32, one column block: 60 calls 1.009 times as long with scalar bases, up to 1.09; one row and two column
    blocks 1.009 and up to 1.18: 5^4 x 205350 x 5 at R = 25, fourth mode 1.14 against 1.35 ms; with more MFMAs a step 0.97 in the mean
    of 65 calls, at most 1.08).  fp64 with three row and two column blocks: the registers of the lanes' offsets lie in scratch memory (8 calls 1.02)."""
    if i.w == 2:
        return i.rb == 3 and i.jb == 2
    return i.jb == 1 or i.rb * i.jb <= 2


def even(n):
    return n + (n & 1)


class Inst:
    def __init__(self, w, rb, jb):
        self.w, self.rb, self.jb = w, rb, jb            # w: registers per value (2 = fp64, 1 = fp32)
        self.xregs = even(rb * w)
        self.bregs = even(jb * w)
        self.set = self.xregs + self.bregs
        self.bc = even(jb * w)
        self.acc = rb * jb * 4 * w
        self.lane = lane_pointers(self)
        # loads of one step: (destination offset in the set, registers, which pointer, byte offset)
        self.xloads = []
        if w == 2:
            if rb in (2, 4):                             # one 8-byte load per row block
                self.xloads = [(2 * r, 2, "xo0", 128 * r) for r in range(rb)]
            elif rb == 1:
                self.xloads = [(0, 2, "xo0", 0)]
            else:                                        # rb == 3: rows 2m, 2m+1 then row 32 + m
                self.xloads = [(0, 4, "xo0", 0), (4, 2, "xo1", 0)]
            g = 2
        else:
            self.xloads = [(0, rb, "xo0", 0)]
            g = 4
        n0 = min(jb, g)
        n1 = jb - n0
        self.bloads = [(0, n0 * w, "bo0")]
        if n1:
            self.bloads.append((n0 * w, n1 * w, "bo1"))
        self.two_x = any(p == "xo1" for _, _, p, _ in self.xloads)
        self.two_b = n1 > 0
        self.loads = len(self.xloads) + len(self.bloads)
        self.pick()

    def ring(self, d):
        return self.set * (d + 1) + self.bc

    def pick(self):
        for budget, waves in ((128, 4), (168, 3), (256, 2)):
            for d in range(D_MAX, D_MIN - 1, -1):
                if d * self.loads > 63:
                    continue
                if self.acc + others(self) + self.ring(d) <= budget:
                    self.budget, self.waves, self.d = budget, waves, d
                    self.t0 = budget - self.ring(d)
                    self.t0 -= self.t0 & 1
                    return
        self.budget = 0      # nothing fits: no pipelined run for this instantiation

    def tag(self):
        return "%s%d%d" % ("d" if self.w == 2 else "f", self.rb, self.jb)

    def ctype(self):
        return "double" if self.w == 2 else "float"

    # --- registers
    def reg(self, base, n):
        return "v%d" % base if n == 1 else "v[%d:%d]" % (base, base + n - 1)

    def xbase(self, s):
        return self.t0 + self.set * s

    def xval(self, s, r):
        return self.reg(self.xbase(s) + r * self.w, self.w)

    def bval(self, s, j):
        return self.reg(self.xbase(s) + self.xregs + j * self.w, self.w)

    def bcval(self, j):
        return self.reg(self.t0 + self.set * (self.d + 1) + j * self.w, self.w)

    def last_reg(self):
        return self.t0 + self.ring(self.d) - 1

    # --- code
    def issue(self, s, nt):
        o = []
        width = {1: "dword", 2: "dwordx2", 3: "dwordx3", 4: "dwordx4"}
        for off, n, lane, byte in self.xloads:
            addr = "%%[%s], off" % lane.replace("xo", "xp") if self.lane else "%%[%s], %s" % (lane, XB)
            o.append("global_load_%s %s, %s%s%s" % (width[n], self.reg(self.xbase(s) + off, n), addr, " offset:%d" % byte if byte else "", nt))
        for off, n, lane in self.bloads:
            o.append("global_load_%s %s, %%[%s], %s" % (width[n], self.reg(self.xbase(s) + self.xregs + off, n), lane, "%[bb]" if self.lane else BB))
        if self.lane:
            for p in ("xp0", "xp1")[:2 if self.two_x else 1]:
                o.append("v_lshl_add_u64 %%[%s], %%[%s], 0, %%[xs]" % (p, p))
            for p in ("bo0", "bo1")[:2 if self.two_b else 1]:
                o.append("v_add_u32 %%[%s], %%[bs], %%[%s]" % (p, p))
            return o
        o.append("s_add_u32 s%d, s%d, s%d" % (S0, S0, S0 + 2))
        o.append("s_addc_u32 s%d, s%d, s%d" % (S0 + 1, S0 + 1, S0 + 3))
        o.append("s_add_u32 s%d, s%d, %%[bs]" % (S0 + 4, S0 + 4))
        o.append("s_addc_u32 s%d, s%d, 0" % (S0 + 5, S0 + 5))
        return o

    def consume(self, s, wait):
        mul = "v_mul_f64" if self.w == 2 else "v_mul_f32"
        mfma = "v_mfma_f64_16x16x4_f64" if self.w == 2 else "v_mfma_f32_16x16x4_f32"
        o = ["s_waitcnt vmcnt(%d)" % wait]
        for j in range(self.jb):
            o.append("%s %s, %s, %%[q%d]" % (mul, self.bcval(j), self.bval(s, j), j))
        o.append("s_nop 1")
        for r in range(self.rb):
            for j in range(self.jb):
                a = "%%[a%d%d]" % (r, j)
                o.append("%s %s, %s, %s, %s" % (mfma, a, self.xval(s, r), self.bcval(j), a))
        return o

    def block(self, nt):
        d, s_n, l = self.d, self.d + 1, self.loads
        o = ["s_nop 4"]
        if not self.lane:
            o += ["s_mov_b64 %s, %%[xb]" % XB, "s_mov_b64 s[%d:%d], %%[xs]" % (S0 + 2, S0 + 3), "s_mov_b64 %s, %%[bb]" % BB]
        for k in range(d):
            o += self.issue(k, nt)
        o.append("1:")
        for u in range(s_n):
            o.append("s_cmp_eq_u32 %[n], 0")
            o.append("s_cbranch_scc1 %df" % (10 + u))
            o += self.issue((u + d) % s_n, nt)
            o.append("s_sub_u32 %[n], %[n], 1")
            o += self.consume(u, d * l)
        o.append("s_branch 1b")
        for u in range(s_n):
            o.append("%d:" % (10 + u))
            for k in range(d):
                o += self.consume((u + k) % s_n, (d - 1 - k) * l)
            if u < s_n - 1:
                o.append("s_branch 9f")
        o.append("9:")
        o += ["s_nop 7", "s_nop 7", "s_nop 7"]
        return o

    def emit(self):
        t = self.tag().upper()
        c = self.ctype()
        out = "// %s: RB = %d, JB = %d; %d steps in flight, ring of %d sets in v[%d:%d], %d wavefronts per SIMD\n" % (
            c, self.rb, self.jb, self.d, self.d + 1, self.t0, self.last_reg(), self.waves)
        flavours = [("", "")] + ([("_NT", " nt")] if self.w == 2 else [])
        for suffix, nt in flavours:
            out += "#define MTTKRP_PIPE_%s_ASM%s \\\n" % (t, suffix)
            out += " \\\n".join('    "%s\\n"' % line for line in self.block(nt)) + "\n"
        clob = ", ".join('"v%d"' % v for v in range(self.t0, self.last_reg() + 1))
        if not self.lane:
            clob += ", " + ", ".join('"s%d"' % v for v in range(S0, S0 + 6))
        accs = ", ".join('[a%d%d] "+v"(acc[%d][%d])' % (r, j, r, j) for r in range(self.rb) for j in range(self.jb))
        lanes = ["%so%d" % (a, n) for a, two in (("x", self.two_x), ("b", self.two_b)) for n in range(2 if two else 1)]
        outs = '[n] "+&s"(n_more), ' + accs
        ins = '[xs] "s"(x_step_bytes), [bb] "s"(bbase), [bs] "s"(b_step_bytes), ' + ", ".join('[q%d] "v"(q[%d])' % (j, j) for j in range(self.jb))
        if self.lane:
            outs = "".join('[%s] "+&v"(%s), ' % (v, v) for v in (a.replace("xo", "xp") for a in lanes)) + outs
        else:
            ins = '[xb] "s"(xp0), ' + "".join('[%s] "v"(%s), ' % (v, v) for v in lanes) + ins
        out += "template <> struct Pipe<%s, %d, %d> {\n" % (c, self.rb, self.jb)
        out += "    static constexpr bool value = true;\n"
        out += "    static constexpr int depth = %d;\n    static constexpr int waves = %d;\n" % (self.d, self.waves)
        out += "    static constexpr bool lane = %s;\n" % ("true" if self.lane else "false")
        out += "    template <bool NT>\n"
        out += "    static __device__ __forceinline__ void run(typename Mfma<%s>::acc_t (&acc)[%d][%d], const %s*%s xp0,\n" % (
            c, self.rb, self.jb, c, "&" if self.lane else "")
        out += "                                               %s, int64_t x_step_bytes, const %s* bbase,\n" % (
            "const %s* xp1" % c if self.lane else "uint32_t xo0, uint32_t xo1", c)
        out += "                                               uint32_t bo0, uint32_t bo1, uint32_t b_step_bytes,\n"
        out += "                                               const %s (&q)[%d], int n_more)\n    {\n" % (c, self.jb)
        if not self.two_x:
            out += "        (void)%s;\n" % ("xp1" if self.lane else "xo1")
        if not self.two_b:
            out += "        (void)bo1;\n"
        if self.w == 2:
            out += "        if (NT)\n"
            out += "            asm volatile(MTTKRP_PIPE_%s_ASM_NT : %s : %s : %s, \"scc\", \"memory\");\n" % (t, outs, ins, clob)
            out += "        else\n    "
        out += "        asm volatile(MTTKRP_PIPE_%s_ASM : %s : %s : %s, \"scc\", \"memory\");\n" % (t, outs, ins, clob)
        out += "    }\n};\n\n"
        return out


def main(path=None):
    """Writes the include file (next to this script unless a path is given) and returns its path."""
    insts = [Inst(w, rb, jb) for w in (2, 1) for rb in (1, 2, 3, 4) for jb in (1, 2, 3, 4)]
    insts = [i for i in insts if i.budget]
    out = "// Generated by gen_pipe.py; do not edit.\n"
    out += "// Primary template: no pipelined run for an instantiation (the kernel then uses batches only).\n"
    out += "template <typename T, int RB, int JB> struct Pipe {\n"
    out += "    static constexpr bool value = false;\n    static constexpr int depth = 1 << 30;\n"
    out += "    static constexpr int waves = 0;\n    static constexpr bool lane = false;\n"
    out += "    template <bool NT>\n"
    out += "    static __device__ __forceinline__ void run(typename Mfma<T>::acc_t (&)[RB][JB], const T*, uint32_t, uint32_t, int64_t,\n"
    out += "                                               const T*, uint32_t, uint32_t, uint32_t, const T (&)[JB], int)\n    {\n    }\n};\n\n"
    for i in insts:
        out += i.emit()
    if path is None:
        path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "mttkrp_pipe.inc")
    with open(path, "w") as f:
        f.write(out)
    for i in insts:
        print("%s: acc %3d, set %2d, depth %d, budget %d (%d waves), ring v[%d:%d], loads/step %d" % (
            i.tag(), i.acc, i.set, i.d, i.budget, i.waves, i.t0, i.last_reg(), i.loads))
    return path


if __name__ == "__main__":
    print(main())
