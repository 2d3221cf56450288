#!/usr/bin/env python3
"""Writes fea_sweep_core.inc: the hand-scheduled gfx950 instruction sequences with which the
waves of one workgroup sweep a piece of a shared run together.
Run it after changing the schedule:  python3 gen_sweep_core.py > fea_sweep_core.inc

A piece of a shared run (one KV head x a range of whole 32-token tiles) is swept for several row
tiles of up to 64 query rows (requests x group heads).  The row tiles read the same KV bytes, so
the planner puts them on neighbouring waves of one workgroup - a team of 2 or of 4 - and the
team fetches every tile once: each wave requests its part of the tile (global -> LDS), the
tiles sit in a ring all team members read, and one workgroup barrier per tile says both "every
part of the next tile has landed" and "everybody is done with the slot about to be refilled".
What a wave computes for its own row tile is what sweep_item computes - per query row the
triple (m, l, acc[128]) of an online softmax over the piece, the reference exponent m raised
(and O^T, l rescaled) only when a score exceeds it by more than 2^24.

Why by hand: a wave has no second wave on its SIMD, so the matrix core only stays busy if the
products of tile t+1 are in flight while the vector unit turns tile t's scores into weights,
and the 240 accumulation registers must stay put for the whole sweep.  The compiler does
neither for this loop (it moves or spills the accumulators), so the registers are assigned
here and the instruction streams - matrix core, vector unit, scalar unit with the memory
requests - are interleaved in program order.

Team of T waves (T = 2, 4), ring of D = 2 T tiles: K ring (D slots of two 4 KB blocks), then V
ring.  Rank r requests, per tile, T = 4: one block (K b0, K b1, V b0, V b1 for r = 0..3, 4
loads); T = 2: both blocks of K (r = 0) or of V (r = 1), 8 loads.  Tiles 0 .. D-1 are requested
up front.  Iteration t: first phase (S of tile t+1, weights of tile t) on K fragments read from LDS
during the iteration before, while V of tile t is read; then, tile t being read out, the barrier, tile
t+D requested into its slot and the K reads of tile t+2 requested, under the second phase's products
(O^T += V^T P^T).  A wave's own requests complete in order, so "my part of tile t+2 has landed" is
vmcnt(loads x min(D-3, n-3-t)).

What bounds an iteration is what one wave issues and fetches: an instruction in four cycles, and 32
bytes of instructions in 19 to 29 cycles, by compute unit (measured with dependent chains: 8-byte
instructions 4.65 cycles apiece at best, 7.2 at worst).  So instructions are what is saved: the scores
sit in vector registers, where the vector unit reads them as they are (in accumulation registers each
is copied out twice, 64 instructions a tile), and V comes out of LDS already transposed
(ds_read_b64_tr_b16: 8 reads more, 32 permutes and their waits less).  The matrix core takes its operands
from accumulation registers as well, so that is where q and the K fragments went instead.  Instructions of
500 requests on one prefix of 10240 tokens 43.0 -> 31.4 million, wave cycles 77 -> 62; 26 shapes with
teams (24 to 300 requests on 600 to 12000 tokens) 0.94 of a call's time in the mean, 0.76 at best.

ds_read_b64_tr_b16: the 16 lanes of a group read four rows of 16 values, lane j four of them in row j / 4;
lane n is left with value n of each of the four rows, which makes it, for 16 dims, the A operand of the
second product as the weights' layout wants it (k-slots: the lane group's 4 tokens in each block).

Register map (fixed, listed as clobbers so that the compiler keeps its own values elsewhere):
  a[0:127]    O^T accumulators   O(nt, i) = a[(8 nt + i) 4 ..]      nt: row tile of 16, i: dims 16 i + 4 kg + jj
  a[128:143]  row sums           L(nt)
  a[144:207]  Q^T fragments      Q(nt, ks)
  a[208:239]  K fragments of the next tile   KA(mt, ks)
  v[32:35] / v[36:43] LDS addresses of this iteration's K / V fragments, v[44:47] / v[48:55] in slot 0
  v[56:87] S^T buffer A, v[88:119] S^T buffer B    S(nt, mt): tokens 16 mt + 4 kg + jj, row 16 nt + n
  v[120:151]  V^T of this tile               VA(i)
  v[152:167]  weights                        P(nt)
  v[168:183]  temporaries, v[184:187] ones, v[188:191] -m per row tile, v[192:195] lane offsets of the loads,
  v196, v[198:199] table address and block ids, v200, v201 lane addresses of the two cross-lane maxima,
  v[202:205] raw score maximum of the coming tile per row tile, v[206:209] scratch.
  s[64:75]    counters, block ids, addresses; s[76:77] exec at the end.
"""

SLOT = 8192           # two blocks of K (or V): one ring slot


def tup(f, b, n=4): return f"{f}[{b}:{b + n - 1}]"
def Q(nt, ks): return tup("a", 144 + (nt * 4 + ks) * 4)
def KA(mt, ks): return tup("a", 208 + (mt * 4 + ks) * 4)
def KBT(ks): return f"v{32 + ks}"      # this iteration's slot
def VBT(i): return f"v{36 + i}"
def KB(ks): return f"v{44 + ks}"       # slot 0
def VB(i): return f"v{48 + i}"
def S(buf, nt, mt): return tup("v", 56 + 32 * buf + (nt * 2 + mt) * 4)
def Se(buf, nt, x): return f"v{56 + 32 * buf + nt * 8 + x}"
def VA(i): return tup("v", 120 + 4 * i)
def VAh(i, blk): return tup("v", 120 + 4 * i + 2 * blk, 2)
def P(nt): return tup("v", 152 + 4 * nt)
def Pe(nt, c): return f"v{152 + 4 * nt + c}"
def T(x): return f"v{168 + x}"
ONES = "v[184:187]"
def NEGM(nt): return f"v{188 + nt}"
def DOFF(q): return f"v{192 + q}"
VTAB, VID, VID0, VID1 = "v196", "v[198:199]", "v198", "v199"
A16, A32 = "v200", "v201"
def TM(nt): return f"v{202 + nt}"
ML, ML0, ML1, VROW, VDST = "v[206:207]", "v206", "v207", "v208", "v209"
def O(nt, i): return tup("a", (nt * 8 + i) * 4)
def LACC(nt): return tup("a", 128 + 4 * nt)

ST, SRING, SB0, SB1, SLO, SHI, STMP, SJ, STMP2 = "s64", "s65", "s68", "s69", "s70", "s71", "s73", "s75", "s74"
SADDR = "s[70:71]"
SEXEC = "s[76:77]"
LAST_V, LAST_A, LAST_S = 209, 239, 77   # registers in use end here


class Gen:
    def __init__(self, team):
        self.T = team
        self.D = 2 * team
        self.L = 4 if team == 4 else 8       # loads per tile part
        self.out = []
        self.uid = 0

    def emit(self, s): self.out.append(s)

    def label(self, stem):
        self.uid += 1
        return f"{stem}{self.uid}_%="

    # ---- memory side
    def table_entry(self, clamped):
        """Lines that ask for the block ids of this wave's part of tile SJ (or the last tile, if that comes before)."""
        v = [f"s_add_u32 {STMP}, %[ntiles], -1", f"s_min_i32 {STMP}, {STMP}, {SJ}"] if clamped else [f"s_mov_b32 {STMP}, {SJ}"]
        v.append(f"s_lshl_b32 {STMP}, {STMP}, 3")
        v.append(f"s_add_u32 {STMP}, {STMP}, %[tab]")
        v.append(f"s_add_u32 {STMP}, {STMP}, %[tabsel]")
        v.append(f"v_mov_b32 {VTAB}, {STMP}")
        v.append(f"ds_read_b32 {VID0}, {VTAB}" if self.T == 4 else f"ds_read_b64 {VID}, {VTAB}")
        return v

    def block_ids(self):
        return [f"v_readfirstlane_b32 {SB0}, {VID0}"] + ([f"v_readfirstlane_b32 {SB1}, {VID1}"] if self.T == 2 else [])

    def requests(self):
        """Lines that request this wave's part of tile SJ, whose block ids are in SB0, SB1.  The immediate offset of a load
        moves both its addresses, so the four loads of a block share one M0."""
        v = [f"s_and_b32 {STMP}, {SJ}, {self.D - 1}", f"s_lshl_b32 {STMP}, {STMP}, 13", f"s_add_u32 m0, {STMP}, {SRING}"]
        for blk, sb in enumerate((SB0, SB1)[: (1 if self.T == 4 else 2)]):
            v.append(f"s_max_i32 {sb}, {sb}, 0")
            v.append(f"s_mul_i32 {STMP}, {sb}, %[hkv]")
            v.append(f"s_add_u32 {STMP}, {STMP}, %[g]")
            v.append(f"s_lshr_b32 {SHI}, {STMP}, 20")
            v.append(f"s_lshl_b32 {SLO}, {STMP}, 12")
            v.append(f"s_add_u32 {SLO}, {SLO}, %[own_lo]")
            v.append(f"s_addc_u32 {SHI}, {SHI}, %[own_hi]")
            if blk == 1:
                v.append("s_addk_i32 m0, 0x1000")
                v.append("s_nop 0")
            # (A team reads every tile once and has it pass by the caches, also where another team reads it too: 40 requests in
            # each of 4 groups behind a system prompt 69.7 -> 67.8 us, 20 in each of 6 60.2 -> 62.8, 500 on one prefix the same;
            # and two forms of the sequence, chosen by the item, cost every team 0.3 us.  32 requests on one of 32K 73.4 -> 64.1.)
            for q in range(4):
                v.append(f"global_load_lds_dwordx4 {DOFF(q)}, {SADDR}" + (f" offset:{1024 * q}" if q else "") + " nt")
        return v

    def issue_own(self):
        """Requests this wave's part of tile SJ (the caller has checked SJ < ntiles)."""
        for x in self.table_entry(False) + ["s_waitcnt lgkmcnt(0)"] + self.block_ids() + self.requests(): self.emit(x)

    def wait_younger(self, sreg, kmax):
        """Waits until at most min(kmax, sreg) of this wave's tile parts are still on their way."""
        e = self.emit
        end = self.label("WE")
        labs = {}
        for k in range(kmax, 0, -1):
            labs[k] = self.label("W")
            e(f"s_cmp_ge_i32 {sreg}, {k}")
            e(f"s_cbranch_scc1 {labs[k]}")
        e("s_waitcnt vmcnt(0)")
        e(f"s_branch {end}")
        for k in range(kmax, 0, -1):
            e(f"{labs[k]}:")
            e(f"s_waitcnt vmcnt({k * self.L})")
            if k > 1:
                e(f"s_branch {end}")
        e(f"{end}:")

    # ---- instruction streams of one tile
    def k_reads(self, kb): return [f"ds_read_b128 {KA(mt, ks)}, {kb(ks)} offset:{mt * 4096}" for mt in range(2) for ks in range(4)]

    def v_reads(self): return [f"ds_read_b64_tr_b16 {VAh(i, blk)}, {VBT(i)} offset:{blk * 4096}" for i in range(8) for blk in range(2)]

    @staticmethod
    def scores(buf):
        """S(buf) = K Q^T for the tile whose K fragments are in KA."""
        return [f"v_mfma_f32_16x16x32_bf16 {S(buf, nt, mt)}, {KA(mt, ks)}, {Q(nt, ks)}, {'0' if ks == 0 else S(buf, nt, mt)}"
                for mt in range(2) for ks in range(4) for nt in range(4)]

    @staticmethod
    def weights_chain(buf, nt):
        """P(nt) = bf16(exp2(S(buf, nt) * scale - m)) for this lane's 8 tokens."""
        t = lambda x: T(8 * (nt & 1) + x)
        return ([f"v_fma_f32 {t(x)}, {Se(buf, nt, x)}, %[scale], {NEGM(nt)}" for x in range(8)] +
                [f"v_exp_f32 {t(x)}, {t(x)}" for x in range(8)] +
                [f"v_cvt_pk_bf16_f32 {Pe(nt, c)}, {t(2 * c)}, {t(2 * c + 1)}" for c in range(4)])

    @staticmethod
    def pv(nt):
        return ([f"v_mfma_f32_16x16x32_bf16 {LACC(nt)}, {ONES}, {P(nt)}, {LACC(nt)}"] +
                [f"v_mfma_f32_16x16x32_bf16 {O(nt, i)}, {VA(i)}, {P(nt)}, {O(nt, i)}" for i in range(8)])

    def addresses(self, tiles_on, cur, base, n):
        """LDS addresses of the fragments in the slot of tile t + tiles_on."""
        v = [f"s_add_u32 {STMP2}, {ST}, {tiles_on}"] if tiles_on else [f"s_mov_b32 {STMP2}, {ST}"]
        v += [f"s_and_b32 {STMP2}, {STMP2}, {self.D - 1}", f"s_lshl_b32 {STMP2}, {STMP2}, 13"]
        return v + [f"v_add_u32 {cur(x)}, {STMP2}, {base(x)}" for x in range(n)]

    def weave(self, products, others, first=0):
        """The products with the other instructions dealt out evenly behind them, from product `first` on."""
        done, slots = 0, len(products) - first
        for k, line in enumerate(products):
            self.emit(line)
            upto = len(others) * (k + 1 - first) // slots if k >= first else 0
            for x in others[done:upto]: self.emit(x)
            done = max(done, upto)

    @staticmethod
    def deal(a, b):
        """Two lists as one, each in its order, evenly mixed."""
        out, j = [], 0
        for k, x in enumerate(a):
            out.append(x)
            upto = len(b) * (k + 1) // len(a)
            out += b[j:upto]
            j = max(j, upto)
        return out

    def tile(self, cur, last, name):
        """Iteration t: weights of tile t from S(cur), O^T += V(t)^T P^T and, unless `last`, S(1-cur) = K(t+1) Q^T.
        K(t+1) was asked for by the iteration before (or the prologue), which has also set the addresses of V(t)."""
        e = self.emit
        nxt = 1 - cur
        D = self.D
        e(f"; ---- {name}")
        chains = self.weights_chain(cur, 0) + self.weights_chain(cur, 1)
        # ---- phase 1
        e("s_waitcnt lgkmcnt(0)")                      # K(t+1)
        if last:
            for x in self.v_reads() + chains: e(x)
            e("s_waitcnt lgkmcnt(0)")
        else:
            memory = self.v_reads() + [f"s_add_u32 {SJ}, {ST}, {D}"] + self.table_entry(True)
            self.weave(self.scores(nxt), self.deal(chains, memory))
            e("s_waitcnt lgkmcnt(0)")
            for x in self.block_ids(): e(x)
            # ---- tile t is read out by me.  My part of tile t+2 has landed; after the barrier everybody's has, and
            # everybody is done with tile t: refill its slot with tile t+D, and ask for K(t+2) (where there is none, what
            # the slot holds is read and not used).
            e(f"s_sub_i32 {STMP}, %[ntiles], {ST}")
            e(f"s_sub_i32 {STMP}, {STMP}, 3")
            self.wait_younger(STMP, D - 3)
            e("s_barrier")
        # ---- phase 2: O^T += V^T P^T for row tiles 0, 1 with the weights of row tile 2 on the vector unit
        e("s_nop 1")
        chain2 = self.weights_chain(cur, 2)
        products = self.pv(0) + self.pv(1)
        if last:
            self.weave(products, chain2)
        else:
            reads = self.addresses(2, KBT, KB, 4) + self.k_reads(KBT)
            no, done = self.label("NI"), self.label("DI")
            e(f"s_cmp_lt_i32 {SJ}, %[ntiles]")
            e(f"s_cbranch_scc0 {no}")
            self.weave(products, self.requests() + self.deal(chain2, reads))
            e(f"s_branch {done}")
            e(f"{no}:")
            self.weave(products, self.deal(chain2, reads))
            e(f"{done}:")
        # ---- phase 3: row tile 2 with the weights of row tile 3; row tile 3 while it is looked whether a score of tile
        # t+1 outgrows its row's reference
        e("s_nop 1")
        self.weave(self.pv(2), self.weights_chain(cur, 3))
        e("s_nop 1")
        check = []
        if not last:
            for nt in range(4):
                a, b = T(2 * (nt & 1)), T(2 * (nt & 1) + 1)
                s = lambda x: Se(nxt, nt, x)
                check.append(f"v_max3_f32 {a}, {s(0)}, {s(1)}, {s(2)}")
                check.append(f"v_max3_f32 {b}, {s(3)}, {s(4)}, {s(5)}")
                check.append(f"v_max3_f32 {a}, {a}, {s(6)}, {s(7)}")
                check.append(f"v_max_f32 {TM(nt)}, {a}, {b}")
                check.append(f"v_fma_f32 {T(4 + nt)}, {TM(nt)}, %[scale], {NEGM(nt)}")
            check += self.addresses(1, VBT, VB, 8)
            check.append(f"v_max3_f32 {T(4)}, {T(4)}, {T(5)}, {T(6)}")
            check.append(f"v_max_f32 {T(4)}, {T(4)}, {T(7)}")
            check.append(f"v_cmp_lt_f32 vcc, 0x41c00000, {T(4)}")
        self.weave(self.pv(3), check)
        if not last:
            no = self.label("NR")
            e(f"s_cbranch_vccz {no}")
            self.raise_refs()
            e(f"{no}:")

    def raise_refs(self):
        """Rare: every row's reference becomes max(old reference, row maximum of the coming tile); O^T and the
        row sums are scaled by 2^(old - new) (1 where nothing changed)."""
        e = self.emit
        e("s_nop 7")
        e("s_nop 7")
        e("s_nop 3")
        for nt in range(4):
            e(f"ds_bpermute_b32 {T(8)}, {A16}, {TM(nt)}")
            e("s_waitcnt lgkmcnt(0)")
            e(f"v_max_f32 {T(9)}, {TM(nt)}, {T(8)}")
            e("s_nop 1")
            e(f"ds_bpermute_b32 {T(8)}, {A32}, {T(9)}")
            e("s_waitcnt lgkmcnt(0)")
            e(f"v_max_f32 {T(9)}, {T(9)}, {T(8)}")
            e(f"v_mul_f32 {T(9)}, %[scale], {T(9)}")
            e(f"v_xor_b32 {T(10)}, 0x80000000, {NEGM(nt)}")
            e(f"v_max_f32 {T(9)}, {T(9)}, {T(10)}")
            e(f"v_sub_f32 {T(10)}, {T(10)}, {T(9)}")
            e(f"v_exp_f32 {T(10)}, {T(10)}")
            e(f"v_xor_b32 {NEGM(nt)}, 0x80000000, {T(9)}")
            e("s_nop 1")
            regs = [f"a{(nt * 8 + i) * 4 + jj}" for i in range(8) for jj in range(4)] + [f"a{128 + 4 * nt + jj}" for jj in range(4)]
            for k in range(0, len(regs), 4):
                grp = regs[k:k + 4]
                for x, r in enumerate(grp): e(f"v_accvgpr_read_b32 {T(11 + x)}, {r}")
                for x, r in enumerate(grp): e(f"v_mul_f32 {T(11 + x)}, {T(10)}, {T(11 + x)}")
                for x, r in enumerate(grp): e(f"v_accvgpr_write_b32 {r}, {T(11 + x)}")
        e("s_nop 7")

    def build(self):
        e = self.emit
        D = self.D
        vring = D * SLOT
        e(f"; ---- team of {self.T}: setup (ones, per-lane addresses)")
        for k in range(4):
            e(f"v_mov_b32 v{184 + k}, 0x3f803f80")
        e(f"s_add_u32 {SRING}, %[team], %[own_ring]")
        e(f"v_add_u32 {KB(0)}, %[team], %[koff0]")
        for ks in range(1, 4):
            e(f"v_xor_b32 {KB(ks)}, {64 * ks}, %[koff0]")
            e(f"v_add_u32 {KB(ks)}, %[team], {KB(ks)}")
        for i in range(8):
            e(f"v_xor_b32 {VB(i)}, {32 * i}, %[voff0]")
            e(f"v_add_u32 {VB(i)}, {vring}, {VB(i)}")
            e(f"v_add_u32 {VB(i)}, %[team], {VB(i)}")
        for i in range(4):
            e(f"v_xor_b32 {DOFF(i)}, {64 * i}, %[doff0]")
        e("; ---- query rows (rows past the end repeat a valid one), then my parts of the first D tiles")
        for nt in range(4):
            for ks in range(4):
                e(f"global_load_dwordx4 {Q(nt, ks)}, %[q{nt}], %[qbase] offset:{64 * ks}")
        for j in range(D):
            no = self.label("NP")
            e(f"s_mov_b32 {SJ}, {j}")
            if j >= 4:
                e(f"s_cmp_lt_i32 {SJ}, %[ntiles]")
                e(f"s_cbranch_scc0 {no}")
            self.issue_own()
            e(f"{no}:")
        for k in range(144):
            e(f"v_accvgpr_write_b32 a{k}, 0")
        e("; ---- S(A) = K(0) Q^T, reference exponent = row maximum of the first tile")
        e(f"s_sub_i32 {STMP}, %[ntiles], 2")       # my parts of tiles 0 and 1
        self.wait_younger(STMP, D - 2)
        e("s_barrier")
        for x in self.k_reads(KB): e(x)
        e("s_waitcnt lgkmcnt(0)")
        for x in self.scores(0): e(x)
        e("s_nop 7")
        e("s_nop 7")
        e(f"v_xor_b32 {A16}, 64, %[lane4]")       # lane ^ 16
        e(f"v_xor_b32 {A32}, 128, %[lane4]")      # lane ^ 32
        for nt in range(4):
            s = lambda x: Se(0, nt, x)
            e(f"v_max3_f32 {T(8)}, {s(0)}, {s(1)}, {s(2)}")
            e(f"v_max3_f32 {T(9)}, {s(3)}, {s(4)}, {s(5)}")
            e(f"v_max3_f32 {T(8)}, {T(8)}, {s(6)}, {s(7)}")
            e(f"v_max_f32 {T(8)}, {T(8)}, {T(9)}")
            e(f"ds_bpermute_b32 {T(10)}, {A16}, {T(8)}")
            e("s_waitcnt lgkmcnt(0)")
            e(f"v_max_f32 {T(8)}, {T(8)}, {T(10)}")
            e("s_nop 1")
            e(f"ds_bpermute_b32 {T(10)}, {A32}, {T(8)}")
            e("s_waitcnt lgkmcnt(0)")
            e(f"v_max_f32 {T(8)}, {T(8)}, {T(10)}")
            e(f"v_mul_f32 {T(8)}, %[scale], {T(8)}")
            e(f"v_max_f32 {T(8)}, 0xff7fffff, {T(8)}")   # (scores of -inf alone: the lowest finite number, see kLowest)
            e(f"v_xor_b32 {NEGM(nt)}, 0x80000000, {T(8)}")
        e(f"s_mov_b32 {ST}, 0")
        for x in self.addresses(1, KBT, KB, 4) + self.k_reads(KBT) + self.addresses(0, VBT, VB, 8): e(x)   # K(1), and where V(0) is
        e("LOOP_%=:")
        e(f"s_add_u32 {STMP}, {ST}, 1")
        e(f"s_cmp_eq_u32 {STMP}, %[ntiles]")
        e("s_cbranch_scc1 LASTA_%=")
        self.tile(0, False, "TA")
        e(f"s_add_u32 {ST}, {ST}, 1")
        e(f"s_add_u32 {STMP}, {ST}, 1")
        e(f"s_cmp_eq_u32 {STMP}, %[ntiles]")
        e("s_cbranch_scc1 LASTB_%=")
        self.tile(1, False, "TB")
        e(f"s_add_u32 {ST}, {ST}, 1")
        e("s_branch LOOP_%=")
        e("LASTA_%=:")
        self.tile(0, True, "LA")
        e("s_branch DONE_%=")
        e("LASTB_%=:")
        self.tile(1, True, "LB")
        e("DONE_%=:")
        e("; ---- partial rows: acc[128] per row as the other sweeps lay them out, then (m, l)")
        e("s_nop 7")
        e("s_nop 7")
        e("s_nop 3")
        e(f"s_mov_b64 {SEXEC}, exec")
        e(f"v_lshlrev_b32 {TM(0)}, 3, %[nrow]")         # (m, l) offset of row n: 8 n
        for nt in range(4):
            e(f"s_mov_b64 exec, {SEXEC}")               # (the (m, l) store of the row tile before narrowed it)
            e(f"v_add_u32 {VROW}, {16 * nt}, %[nrow]")
            e(f"v_cmp_gt_i32 vcc, %[nrows], {VROW}")
            e(f"s_and_b64 exec, {SEXEC}, vcc")
            e(f"v_add_u32 {VDST}, {16 * nt * 512}, %[dst0]")
            for i in range(8):
                e(f"global_store_dwordx4 {VDST}, {O(nt, i)}, %[accbase]" + (f" offset:{64 * i}" if i else ""))
            e(f"v_xor_b32 {ML0}, 0x80000000, {NEGM(nt)}")
            e(f"v_accvgpr_read_b32 {ML1}, a{128 + 4 * nt}")
            e(f"v_cmp_gt_u32 vcc, 64, %[lane4]")          # (m, l): lanes of the first lane group only
            e(f"s_and_b64 exec, exec, vcc")
            e(f"v_add_u32 {TM(1)}, {16 * nt * 8}, {TM(0)}")
            e("s_nop 0")
            e(f"global_store_dwordx2 {TM(1)}, {ML}, %[mlbase]")
            e("s_nop 1")
        e(f"s_mov_b64 exec, {SEXEC}")
        e("s_waitcnt vmcnt(0)")
        return self.out


def main():
    print("// Generated by gen_sweep_core.py - do not edit by hand.")
    for team in (2, 4):
        lines = Gen(team).build()
        print(f"#define FEA_TEAM{team}_CORE_ASM \\")
        print(" \\\n".join(f'    "{line}\\n\\t"' for line in lines))
        print()
    vregs = ", ".join(f'"v{k}"' for k in range(32, LAST_V + 1))
    aregs = ", ".join(f'"a{k}"' for k in range(0, LAST_A + 1))
    sregs = ", ".join(f'"s{k}"' for k in range(64, LAST_S + 1))
    print(f"#define FEA_TEAM_CORE_CLOBBERS {vregs}, {aregs}, {sregs}, \"vcc\", \"scc\", \"m0\", \"memory\"")


if __name__ == "__main__":
    main()
