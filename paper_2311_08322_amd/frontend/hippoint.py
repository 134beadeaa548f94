"""Kernels of a fusion group evaluated point by point: the form the generator
uses wherever a group allows it (hipgen.py's staged form serves the rest).

A lane owns one column of a 64 x 4 tile.  Per level the input boxes read at
horizontal offsets go through LDS (double buffered: one barrier per level, none
if nothing is read at an offset), and every temporary is a local of the lane:
one read at an offset is evaluated again at that offset from the inputs
(`_Values`, each value once per level), one that a later computation reads at
its own point stays in a register.  That trades a few operations, which idle
here, for the barriers and LDS passes of staged temporaries.

Loads run PD levels ahead through register rings.  Their addresses are clamped
into the field (a lane or level outside computes values nobody stores), so no
branch stands between a load and its use and the wait counts stay exact.

A temporary that the first sweep writes and only the opposite sweep after it
reads, at the lane's own point (the factors of a tridiagonal solve), need not
go through memory: the column's levels are stashed on chip (`_stash`), the last
written, which are read back first, in registers (the level loop is unrolled
there), those before them in LDS, and only what is left in the workspace.

Measured on the benchmark step, FP64 512x512x80: 325 us with staged
temporaries, one level ahead, and the factors in the workspace (1428 MB moved,
memory bound); 190 us in this form (24 of the 80 levels leave the chip).  Small
domains are bound by the column's serial chain and the barriers in it: 256x256x80
210 -> 66 us, 128x128x40 102 -> 30 us.
"""
from __future__ import annotations

from . import ir

TI, TJ, NT = 64, 4, 256
LDS_BYTES = 160 * 1024
# Levels loaded ahead; 2 is as good while the column stays on chip, 4 wins where
# part of it goes to the workspace (vadv FP64 301x203x137: 105 against 94 us).
PD = 4
# Workspace levels the reading sweep loads ahead (8 against 4: FP32 step
# 512x380x107 125 -> 120 us; 16 the same).
PDW = 8
MAX_LOCALS = 160
# A ring holds PD values of every input; past RING_VALUES inputs it is half as
# deep, past three times that (or boxes beyond a workgroup's share of LDS) the
# group is staged.
RING_VALUES = 8
# The stash by element size: waves per SIMD (workgroups per CU), and the VGPRs a
# lane spends on it.  The column could stay on chip whole at one wave per SIMD,
# but 512x512x80 FP64 then takes 274 us against 199: the second wave hides the
# first's chain.  FP32: 4 waves with 64 VGPRs 106 us, 3 with 96 128 us, 2 with
# 160 126 us.
STASH = {8: (2, 160), 4: (4, 64)}


class Ineligible(Exception):
    """The group needs the staged form."""


def _off(v):
    return f"{'m' if v < 0 else 'p'}{abs(v)}"


def _merge_blocks(prun):
    """The run's PARALLEL computations as (block indices' owner, interval, statements) chains;
    consecutive computations of one block over the same levels become one."""
    out = []
    for cp in prun:
        if out and len(cp.blocks) == 1 and len(out[-1]) == 1 and out[-1][0][1] == cp.blocks[0][0]:
            b, iv, st = out[-1][0]
            out[-1] = [(b, iv, st + tuple(cp.blocks[0][1]))]
            continue
        out.append([((cp.index, bi), iv, tuple(stmts)) for bi, (iv, stmts) in enumerate(cp.blocks)])
    return out


class _Values:
    """Demand-driven evaluation of a PARALLEL block's variables: each (variable,
    version, offset) becomes one local.  A definition is an expression in the
    environment (variable -> version) of its statement ("expr", or "cond" for
    the condition of an if), or a selection by a condition ("sel")."""

    def __init__(self, pk):
        self.pk = pk
        self.defs = []
        self.memo = {}
        self.lines = []

    def _new(self, d):
        self.defs.append(d)
        return len(self.defs) - 1

    def run(self, stmts, env):
        for s in stmts:
            if isinstance(s, ir.Assign):
                env[s.target] = self._new(("expr", s.value, dict(env)))
                continue
            c = self._new(("cond", s.cond, dict(env)))
            et, ee = dict(env), dict(env)
            self.run(s.then, et)
            self.run(s.orelse, ee)
            for n in {**et, **ee}:
                if et.get(n) == ee.get(n):
                    continue
                if n not in et or n not in ee:
                    raise Ineligible(f"{n} is written in one branch only")
                env[n] = self._new(("sel", c, et[n], ee[n]))

    def value(self, v, off):
        key = (v, off)
        if key in self.memo:
            return self.memo[key]
        d = self.defs[v]
        typ = "bool" if d[0] == "cond" else "real"
        if d[0] == "sel":
            c, a, b = (self.value(x, off) for x in d[1:])
            text = f"({c} ? {a} : {b})"
        else:
            if off != (0, 0) and _costly(d[1]):
                raise Ineligible("a costly value is read at an offset")
            text = self.pk.gen.expr(d[1], lambda a: self._access(a, d[2], off))
        var = f"{typ[0]}{v}_{_off(off[0])}{_off(off[1])}"
        self.lines.append(f"const {typ} {var} = ({typ})({text});")
        self.pk.locals += 1
        if self.pk.locals > MAX_LOCALS:
            raise Ineligible("too many values per point")
        self.memo[key] = var
        return var

    def _access(self, a, env, off):
        o = (a.offset[0] + off[0], a.offset[1] + off[1], a.offset[2])
        if a.name in env:
            return self.value(env[a.name], o[:2])
        return self.pk.primitive(a.name, o)


def _costly(e):
    if isinstance(e, ir.Binary) and e.op == "/":
        return True
    if isinstance(e, ir.Builtin) and e.name in ("sqrt", "exp", "log"):
        return True
    return any(_costly(c) for c in ir.expr_children(e))


def _assigned(stmts, top=True):
    """(names assigned by top-level statements, names assigned inside an if)"""
    t, n = set(), set()
    for s in stmts:
        if isinstance(s, ir.Assign):
            (t if top else n).add(s.target)
        else:
            a, b = _assigned(s.then + s.orelse, False)
            n |= a | b
    return t, n


class PointKernel:
    def __init__(self, gen, gi, members):
        self.gen, self.p, self.gi = gen, gen.p, gi
        self.prun = [cp for cp in members if cp.order == ir.PARALLEL]
        self.seqs = [cp for cp in members if cp.order != ir.PARALLEL]
        self.size = 8 if gen.real == "double" else 4
        if self.seqs and self.seqs[0].region != (0, 0, 0, 0):
            raise Ineligible("the sweep runs beyond the domain")
        if not any(f.written for f in self.p.fields.values()):
            raise Ineligible("no output")
        self.pwrites = {n for cp in self.prun for n in cp.writes}
        for n in self.pwrites:
            if n in self.p.temps and self.p.temps[n].storage == "hbm" and self.p.temps[n].ext != (0, 0, 0, 0):
                raise Ineligible(f"{n} leaves the kernel beyond the domain")
        for cp in self.prun:
            for _, stmts in cp.blocks:
                for s in stmts:
                    gen._check_if_offsets(s)
        self.up = not self.seqs or self.seqs[0].order != ir.BACKWARD
        self.chains = _merge_blocks(self.prun)
        self.stash = self._stash()
        # passes until the reads are known (which inputs need boxes, which variables registers)
        self.boxes, self.hoff, self.need_reg = {}, {}, set()
        known = None
        while known != (known := (self.boxes, set(self.need_reg))):
            self.cols, self.locals = [], 0
            self.body = self._par_code() + self._sweep_code()
            self.boxes = {k: (min(o[0] for o in v), max(o[0] for o in v), min(o[1] for o in v), max(o[1] for o in v))
                          for k, v in sorted(self.hoff.items()) if any(o != (0, 0) for o in v)}
        self.values = values = len(self._lead(self.cols)[0]) + sum(self._box(k)[2] for k in self.boxes)
        self.pd = PD if values <= RING_VALUES else PD // 2
        if values > 3 * RING_VALUES or sum(2 * self._box(k)[1] * self.size for k in self.boxes) > LDS_BYTES // 4:
            raise Ineligible("too many inputs in flight")
        self.cols1 = []  # what the sweep that reads the stash loads
        self.body1 = self._second_code(self.seqs[1], self.cols1) if self.stash else []

    # ------------------------------------------------------------ plan
    def _stash(self):
        """Names of the temporaries that stay on chip between the first sweep and
        the opposite one after it."""
        if len(self.seqs) < 2 or self.seqs[1].order == self.seqs[0].order:
            return []
        s0, s1 = self.seqs[:2]
        out = []
        for n in s0.writes:
            t = self.p.temps.get(n)
            if t is None or t.storage != "hbm" or t.comps != {s0.index} or not t.read_comps <= {s0.index, s1.index}:
                continue
            ok = s1.index in t.read_comps
            for _, stmts in s1.blocks:
                for s in stmts:
                    ok &= all(a.offset == (0, 0, 0) for a in ir.stmt_accesses(s)[0] if a.name == n)
            for _, stmts in s0.blocks:
                top, inner = _assigned(stmts)
                ok &= n in top and n not in inner and n not in _read_first(stmts, set(s0.writes))
            if ok:
                out.append(n)
        return out

    def _sizes(self):
        """(waves per SIMD, levels in registers, levels in LDS) of the stash."""
        waves, regs = STASH[self.size]
        # STASH leaves room for rings of the step's size (5 values)
        regs -= max(0, self.values * self.pd - 5 * PD) * self.size // 4
        per = len(self.stash)
        R = max(self.pd, regs * 4 // (per * self.size) // self.pd * self.pd)
        box = sum(2 * self._box(k)[1] * self.size for k in self.boxes)
        NL = max(0, (LDS_BYTES // waves - box - 512) // (per * NT * self.size))
        return waves, R, NL

    def _box(self, key):
        """(width, padded element count, loads per lane) of a box"""
        e = self.boxes[key]
        w, h = TI + e[1] - e[0], TJ + e[3] - e[2]
        it = (w * h + NT - 1) // NT
        return w, it * NT, it

    # ------------------------------------------------------------ level code
    def primitive(self, name, o):
        """A value the level's evaluation does not compute: an input, or a
        variable an earlier computation of the run left in a register."""
        if name in self.pwrites:
            if o != (0, 0, 0) or name not in self.p.temps:
                raise Ineligible(f"{name} read off the lane's point")
            self.need_reg.add(name)
            return f"r_{name}"
        if name in self.p.fields:
            self.hoff.setdefault((name, o[2]), {(0, 0)}).add(o[:2])
            if (name, o[2]) in self.boxes:
                w = self._box((name, o[2]))[0]
                return f"P_{name}_{_off(o[2])}[{o[1] * w + o[0]}]"
            if o[:2] != (0, 0):
                return "(real)0"  # first pass: becomes a box
            return self._col("f", name, o[2])
        if o[:2] != (0, 0) or self.p.temps[name].storage != "hbm":
            raise Ineligible(f"{name} read off the lane's column")
        return self._col("t", name, o[2])

    def _col(self, kind, name, dk):
        if (kind, name, dk) not in self.cols:
            self.cols.append((kind, name, dk))
        return f"x_{kind}_{name}_{_off(dk)}"

    def _store(self, name):
        """Lines storing `v_` as the lane's value of a variable in memory."""
        if name in self.p.fields:
            return [f"if (act) fp_{name}[(int64_t)k * A.f_{name}_sk] = v_;"]
        if self.p.temps[name].storage == "hbm" and name not in self.stash:
            return [f"if (act) tp_{name}[(int64_t)k * A.t_{name}_sk] = v_;"]
        return []

    def _par_code(self):
        out = []
        for chain in self.chains:
            for n, (b, iv, stmts) in enumerate(chain):
                vals, env = _Values(self), {}
                vals.run(stmts, env)
                lines = []
                for name, v in env.items():
                    st = self._store(name)
                    if not st and name not in self.need_reg:
                        continue
                    x = vals.value(v, (0, 0))
                    if name in self.need_reg:
                        lines.append(f"r_{name} = {x};")
                    if st:
                        lines += [f"{{ const real v_ = {x};"] + st + ["}"]
                x = self.gen.bidx[b]
                whole = len(chain) == 1 and iv.start is None and iv.end is None
                cond = "" if whole else f"if (k >= A.blo[{x}] && k < A.bhi[{x}]) "
                out += [f"{'else ' if n else ''}{cond}{{"] + ["  " + l for l in vals.lines + lines] + ["}"]
        return out

    def _sweep_code(self):
        if not self.seqs:
            return []
        cp = self.seqs[0]

        def acc(a):
            if a.name in cp.writes:
                return f"cur_{cp.index}_{a.name}" if a.offset[2] == 0 else f"prev_{cp.index}_{a.name}"
            return self.primitive(a.name, a.offset)
        return self._sweep_level(cp, acc)

    def _sweep_level(self, cp, acc):
        c = cp.index
        out = ["bool done = false;"]
        for bi, (_, stmts) in enumerate(cp.blocks):
            b = self.gen.bidx[(c, bi)]
            out += [f"if (!done && k >= A.blo[{b}] && k < A.bhi[{b}]) {{", "  done = true;"]
            for v in _read_first(stmts, set(cp.writes)):
                if v in self.p.fields:
                    src = f"fp_{v}[(int64_t)k * A.f_{v}_sk]"
                elif self.p.temps[v].storage == "hbm":
                    src = f"tp_{v}[(int64_t)k * A.t_{v}_sk]"
                else:
                    raise Ineligible(f"{v} read before the sweep assigns it")
                out.append(f"  cur_{c}_{v} = act ? {src} : (real)0;")

            def store(name, v):
                return [f"cur_{c}_{name} = {v};"] + self._store(name)
            for s in stmts:
                out += ["  " + l for l in self.gen.stmt_code(s, acc, store)]
            out.append("}")
        if cp.kcache:
            out += ["if (done) {"] + [f"  prev_{c}_{v} = cur_{c}_{v};" for v in cp.kcache] + ["}"]
        return out

    # ------------------------------------------------------------ loads
    def _lead(self, cols):
        """Inputs whose value the previous level held one level on are carried
        over; the others are loaded.  (loaded, {carried: source})"""
        st = 1 if self.up else -1
        carried = {(kd, n, dk): (kd, n, dk + st) for (kd, n, dk) in cols if (kd, n, dk + st) in cols}
        return [c for c in cols if c not in carried], carried

    def _ld(self, key, k):
        kind, name, dk = key
        if kind == "f":
            return f"fp_{name}[(int64_t)kclamp({k} + ({dk}), A.f_{name}_kl, A.f_{name}_kh) * A.f_{name}_sk]"
        return f"tp_{name}[(int64_t)kclamp({k} + ({dk}), 0, A.nk - 1) * A.t_{name}_sk]"

    # ------------------------------------------------------------ kernel
    def source(self):
        p, gi, seqs = self.p, self.gi, self.seqs
        stash = self.stash
        waves, R, NL = self._sizes() if stash else (0, 0, 0)
        pd = self.pd
        bounds = f"__launch_bounds__({NT}, {waves})" if stash else f"__launch_bounds__({NT})"
        I = "__attribute__((always_inline))"
        L = [f"__global__ void {bounds} gts_g{gi}(Args A) {{",
             "  const int tid = threadIdx.x;",
             f"  const int tiles_i = (A.ni + {TI - 1}) / {TI};",
             f"  const int i0 = (int)(blockIdx.x % tiles_i) * {TI}, j0 = (int)(blockIdx.x / tiles_i) * {TJ};",
             f"  const int i = i0 + (tid & {TI - 1}), j = j0 + tid / {TI};",
             "  const bool act = i < A.ni && j < A.nj;",
             "  const int ic = imin(i, A.ni - 1), jc = imin(j, A.nj - 1);"]
        cols1, body1 = self.cols1, self.body1
        # lane pointers
        names = {n for cp in self.prun + seqs for n in cp.writes} | {c[1] for c in self.cols + cols1}
        for f in p.sdef.fields:
            if f in names:
                L.append(f"  real* const fp_{f} = A.f_{f} + (A.f_{f}_any ? (int64_t)ic + (int64_t)jc * A.f_{f}_sj : 0);")
        for t in self.gen.hbm:
            if t.name in names:
                L.append(f"  real* const tp_{t.name} = A.t_{t.name} + ((int64_t)ic + (int64_t)jc * A.t_{t.name}_sj);")
        for key, e in self.boxes.items():
            f, tag = key[0], f"{key[0]}_{_off(key[1])}"
            w, cnt, it = self._box(key)
            n = w * (TJ + e[3] - e[2])
            fe = p.fields[f].ext
            L.append(f"  __shared__ real S_{tag}[{2 * cnt}];")
            L.append(f"  const real* bp_{tag}[{it}];")
            L += ["#pragma unroll", f"  for (int t = 0; t < {it}; ++t) {{",
                  f"    const int el = imin(tid + t * {NT}, {n - 1});",
                  f"    const int gi = imax({fe[0]}, imin(i0 + ({e[0]}) + el % {w}, A.ni + ({fe[1] - 1})));",
                  f"    const int gj = imax({fe[2]}, imin(j0 + ({e[2]}) + el / {w}, A.nj + ({fe[3] - 1})));",
                  f"    bp_{tag}[t] = A.f_{f} + (A.f_{f}_any ? (int64_t)gi + (int64_t)gj * A.f_{f}_sj : 0);", "  }",
                  f"  const int sc_{tag} = ((tid & {TI - 1}) - ({e[0]})) + (tid / {TI} - ({e[2]})) * {w};"]
        if stash:
            for n in stash:
                L.append(f"  real R_{n}[{R}];")
                if NL:
                    L.append(f"  __shared__ real L_{n}[{NL * NT}];")
        for n in sorted(self.need_reg):
            L.append(f"  real r_{n} = (real)0;")
        for cp in seqs:
            L += ["  " + l for l in self.gen.seq_decls(cp)]
        # the level range
        if seqs:
            L.append(f"  const int lo = A.glo[{gi}], hi = A.ghi[{gi}], n = hi - lo;")
        else:
            L.append("  const int lo = blockIdx.y * A.kchunk, hi = imin(lo + A.kchunk, A.nk), n = hi - lo;")
        kof = "lo + ({s})" if self.up else "hi - 1 - ({s})"
        loaded, carried = self._lead(self.cols)
        q = [f"q_{kd}_{n}_{_off(dk)}" for kd, n, dk in loaded]
        for r in q:
            L.append(f"  real {r}[{pd}];")
        for key in self.boxes:
            L.append(f"  real qb_{key[0]}_{_off(key[1])}[{pd}][{self._box(key)[2]}];")
        L += [f"  auto issue = [&](int slot, int s) {I} {{",
              f"    const int k = {kof.format(s='imax(imin(s, n - 1), 0)')};"]
        for r, key in zip(q, loaded):
            L.append(f"    {r}[slot] = {self._ld(key, 'k')};")
        for key in self.boxes:
            f, tag = key[0], f"{key[0]}_{_off(key[1])}"
            L += [f"    const int64_t o_{tag} = (int64_t)kclamp(k + ({key[1]}), A.f_{f}_kl, A.f_{f}_kh) * A.f_{f}_sk;",
                  "#pragma unroll",
                  f"    for (int t = 0; t < {self._box(key)[2]}; ++t) qb_{tag}[slot][t] = bp_{tag}[t][o_{tag}];"]
        L.append("  };")
        L += ["#pragma unroll", f"  for (int s = 0; s < {pd}; ++s) issue(s, s);"]
        for (kd, n, dk) in carried:
            L.append(f"  real h_{kd}_{n}_{_off(dk)} = {self._ld((kd, n, dk), kof.format(s='0'))};")
        # one level
        L += [f"  auto level = [&](int s, int slot, bool more) {I} {{", f"    const int k = {kof.format(s='s')};"]
        for r, (kd, n, dk) in zip(q, loaded):
            L.append(f"    const real x_{kd}_{n}_{_off(dk)} = {r}[slot];")
        # nearest the loaded level last: each reads its source before that moves on
        order = sorted(carried, key=lambda c: c[2], reverse=not self.up)
        for (kd, n, dk) in order:
            L.append(f"    const real x_{kd}_{n}_{_off(dk)} = h_{kd}_{n}_{_off(dk)};")
        for c in order:
            L.append(f"    h_{c[0]}_{c[1]}_{_off(c[2])} = x_{carried[c][0]}_{carried[c][1]}_{_off(carried[c][2])};")
        for key in self.boxes:
            tag = f"{key[0]}_{_off(key[1])}"
            w, cnt, it = self._box(key)
            L += [f"    real* const B_{tag} = S_{tag} + (s & 1) * {cnt};", "#pragma unroll",
                  f"    for (int t = 0; t < {it}; ++t) B_{tag}[tid + t * {NT}] = qb_{tag}[slot][t];"]
        L += [f"    if (more) issue(slot, s + {pd});", '    __asm__ volatile("" ::: "memory");  // the loads stay here']
        if self.boxes:
            L.append("    __syncthreads();")
        for key in self.boxes:
            tag = f"{key[0]}_{_off(key[1])}"
            L.append(f"    const real* const P_{tag} = B_{tag} + sc_{tag};")
        L += ["    " + l for l in self.body]
        L.append("  };")
        if not stash:
            # The last pd levels load nothing ahead, and the loop before them has no
            # branch.  With loads and a check of s < n at every level, short columns
            # were slower than staged (FP64, us, staged, so, now: u * c + v 1000x500x8
            # 17.6, 19.6, 16.6, 512x512x20 24.1, 27.0, 25.0, 838x538x19 40.3, 44.7,
            # 42.7; an upwind difference 1000x500x8 18.0, 20.6, 17.5; a forward sum
            # 384x384x64 56.8, 50.8, 33.6; FP32 33.2, 27.5, 20.6).
            L += ["  int s0 = 0;", f"  for (; s0 + {pd} < n; s0 += {pd}) {{", "#pragma unroll",
                  f"    for (int t = 0; t < {pd}; ++t) level(s0 + t, t, true);", "  }", "#pragma unroll",
                  f"  for (int t = 0; t < {pd}; ++t)", "    if (s0 + t < n) level(s0 + t, t, false);"]
        else:
            c0 = seqs[0].index
            L += [f"  // the stash: levels [nl, n) in registers, [nw, nl) in LDS, [0, nw) in the workspace",
                  f"  const int nl = n > {R} ? (n - {R} + {pd - 1}) / {pd} * {pd} : 0, m = n - nl;",
                  f"  const int nw = imax(nl - {NL}, 0);",
                  f"  for (int s0 = 0; s0 < nl; s0 += {pd}) {{", "#pragma unroll",
                  f"    for (int t = 0; t < {pd}; ++t) {{", "      const int s = s0 + t;", "      level(s, t, true);"]
            lds = [f"L_{n}[(s - nw) * {NT} + tid] = cur_{c0}_{n};" for n in stash] if NL else []
            ws = [f"tp_{n}[(int64_t)({kof.format(s='s')}) * A.t_{n}_sk] = cur_{c0}_{n};" for n in stash]
            L += ["      if (s >= nw) {"] + ["        " + l for l in lds] + ["      } else if (act) {"]
            L += ["        " + l for l in ws] + ["      }", "    }", "  }"]
            L += ["#pragma unroll", f"  for (int r = 0; r < {R}; ++r)", "    if (r < m) {",
                  f"      level(nl + r, r % {pd}, true);"]
            L += [f"      R_{n}[r] = cur_{c0}_{n};" for n in stash] + ["    }"]
            # the opposite sweep
            for (kd, n, dk) in cols1:
                L.append(f"  real y_{kd}_{n}_{_off(dk)} = {self._ld((kd, n, dk), kof.format(s='imax(n - 1, 0)'))};")
            args = ", ".join(f"const real st_{n}" for n in stash)
            L += [f"  auto back = [&](int s, {args}) {I} {{", f"    const int k = {kof.format(s='s')};",
                  f"    const int kn = {kof.format(s='imax(s - 1, 0)')};"]
            for (kd, n, dk) in cols1:
                L.append(f"    const real x_{kd}_{n}_{_off(dk)} = y_{kd}_{n}_{_off(dk)};")
                L.append(f"    y_{kd}_{n}_{_off(dk)} = {self._ld((kd, n, dk), 'kn')};")
            L += ["    " + l for l in body1] + ["  };"]
            L += ["#pragma unroll", f"  for (int r = {R - 1}; r >= 0; --r)",
                  "    if (r < m) back(nl + r, " + ", ".join(f"R_{n}[r]" for n in stash) + ");"]
            if NL:
                L.append("  for (int s = nl - 1; s >= nw; --s) back(s, "
                         + ", ".join(f"L_{n}[(s - nw) * {NT} + tid]" for n in stash) + ");")
            for n in stash:
                L.append(f"  real w_{n}[{PDW}];")
            L += [f"  auto fetch = [&](int slot, int s) {I} {{", f"    const int64_t k = {kof.format(s='imax(s, 0)')};"]
            L += [f"    w_{n}[slot] = tp_{n}[k * A.t_{n}_sk];" for n in stash] + ["  };"]
            L += ["  if (nw > 0) {", "#pragma unroll", f"    for (int t = 0; t < {PDW}; ++t) fetch(t, nw - 1 - t);",
                  f"    for (int t0 = 0; t0 < nw; t0 += {PDW}) {{", "#pragma unroll",
                  f"      for (int t = 0; t < {PDW}; ++t) {{", "        const int s = nw - 1 - t0 - t;"]
            L += [f"        const real a_{n} = w_{n}[t];" for n in stash]
            L += [f"        fetch(t, s - {PDW});", '        __asm__ volatile("" ::: "memory");',
                  "        if (s >= 0) back(s, " + ", ".join(f"a_{n}" for n in stash) + ");", "      }", "    }", "  }"]
        rest = seqs[2:] if stash else seqs[1:]
        L += self.gen.later_sweeps(gi, rest, len(seqs) - len(rest))
        L.append("}")
        return "\n".join(L)

    def _second_code(self, cp, cols):
        """A level of the sweep that reads the stash."""
        def acc(a):
            if a.name in cp.writes:
                return f"cur_{cp.index}_{a.name}" if a.offset[2] == 0 else f"prev_{cp.index}_{a.name}"
            if a.name in self.stash:
                return f"st_{a.name}"
            kind = "f" if a.name in self.p.fields else "t"
            if a.offset[:2] != (0, 0):
                di, dj, dk = a.offset
                if kind == "f":
                    return self.gen.gld_field(a.name, f"i + ({di})", f"j + ({dj})", f"k + ({dk})", "act")
                return self.gen.gld_temp(a.name, f"i + ({di})", f"j + ({dj})", f"k + ({dk})", "act")
            if kind == "t" and self.p.temps[a.name].storage != "hbm":
                raise Ineligible(f"{a.name} read outside its computation")
            key = (kind, a.name, a.offset[2])
            if key not in cols:
                cols.append(key)
            return f"x_{kind}_{a.name}_{_off(a.offset[2])}"
        return self._sweep_level(cp, acc)


def _read_first(stmts, wset):
    """Variables of the sweep read at the current level before it assigns them there."""
    need = []

    def scan(stmts, assigned):
        for s in stmts:
            for a in (ir.accesses(s.value) if isinstance(s, ir.Assign) else ir.accesses(s.cond)):
                if a.name in wset and a.offset[2] == 0 and a.name not in assigned and a.name not in need:
                    need.append(a.name)
            if isinstance(s, ir.Assign):
                assigned.add(s.target)
            else:
                t, e = set(assigned), set(assigned)
                scan(s.then, t)
                scan(s.orelse, e)
                assigned |= t & e
    scan(stmts, set())
    return need
