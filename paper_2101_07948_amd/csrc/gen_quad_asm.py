"""Generates quad_asm_gen.h: the consumer loops of the gfx950 row-group kernel as inline
assembly: one per number of quads of rows a wave holds, NS = 1, 2 (lane groups of 16) and
NS = 4, 8 (lane groups of 4).

A wavefront works on 4 NS rows of W at once over a tile of 64 columns of C.  Its 64 lanes form
groups; one step multiplies one entry of each group's row, so the groups read different B rows
from LDS with the same instruction and no instruction is tied to one row:
  * groups of 16 lanes (NS = 1, 2: one or two sets of four rows): a lane holds 4 columns; a step
    is one ds_read_b128 (16 lanes cover a 256-byte row) and 4 FMAs;
  * groups of 4 lanes (NS = 4, 8: one or two sets of 16 rows): a lane holds 16 columns, four of
    each quarter of the tile; a step is 4 ds_read_b128 and 16 FMAs.  Read i of group g takes
    quarter i ^ (g % 4): the four groups whose lanes LDS serves together then read different
    banks whatever their rows (all reading quarter i, 3.4 cycles of every read's 4.8 went to
    bank conflicts and the layer at 768 x 3072, 90 %, N = 4096 took 113 us instead of 50).
The weight and the LDS address of an entry reach the lanes of its group by a DPP broadcast
(row_newbcast within 16 lanes, quad_perm within 4), so that neither needs a scalar register,
VGPR index mode or a per-entry scalar instruction, and the accumulators are fixed registers.
A DPP instruction takes 4.6 cycles of a SIMD and a plain FMA 3.0, so the groups of 4 move the
weight to a register once per 16 plain FMAs; with groups of 16 one move per 4 FMAs would cost
what it saves, and the FMAs take the broadcast themselves.

Stream consumed (see QuadPacked in sdnn_internal.h): blocks of 64 dwords, one per lane.
Groups of 16: 8 units (8 / NS steps of NS sets, unit u = step * NS + set), lane 16 r + u holds
row r's weight of unit u, lane 16 r + 8 + u its LDS address.  Groups of 4: 2 units (8 / NS
steps of NS / 4 sets), lane 4 r + 2 u holds row r's weight of unit u, lane 4 r + 2 u + 1 its
LDS address.  Descriptors, one dword per sync point:
    c_hi << 19 | c_lo << 6 | n
the next n blocks read chunks c_lo..c_hi only.  n = 0 ends the program, or, with c_lo set
(kQuadMoreDescs), moves on to the next 64 descriptors.  At a sync point the
wave publishes c_lo in its progress word (nothing below it is read again) and waits until
the producers' ready words exceed c_hi.

Register plan (pinned in the asm statement): v[20:23] the stream blocks in flight (four, each
loaded again as soon as it is consumed), v[24:27] the producers' ready words while polling;
else, for groups of 4, v24 and v30 the weights and v[25:27] 64, 128, 192; v28 4 * lane, v29 64
descriptors (one per lane, read with v_readlane), v30 temp, v31 the lane's byte offset in a
B row (with the item's slot flip: the address is the stream's XOR v31), v[32:63] / v[64:95] B values of
the block being multiplied / fetched, v[96:...] accumulators (4 or 16 per set).

Per block g: at the end of a descriptor, the sync point of the next one; addresses and
ds_reads of block g + 1; the FMAs of block g, each quarter of a unit (or the whole block, for
groups of 16) after the reads it needs have landed (LDS returns in order, so lgkmcnt counts
down through them); load block g + 4 into block g's register.  The loads run up to
kQuadTailBlocks blocks past a program's end; the stream carries as many at its end.
A wave's waits are bounded by its poll budget, over all the items it runs; a wave that went on without waiting, or whose chunks a
producer may have overwritten, leaves the NaN POISON in every accumulator, by which the epilogue
knows it.
"""
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "quad_asm_gen.h")

UNITS = 8
WREG = (24, 30)     # weights (groups of 4)
QREG = 25           # v[25:27]: 64, 128, 192 (groups of 4)
EREG = 20           # v[20:23]: stream blocks in flight
NE = 4
VB = (32, 64)
ACC = 96
HISHIFT, LOSHIFT, NBITS = 19, 6, 6
POISON = 0x7FC0DEAD
NMASK = (1 << NBITS) - 1
NSETS = (1, 2, 4, 8)
# SGPRs
PTR, DPTR = 36, 38        # 64-bit
SREADY, STMP, SPOLL, SREADY1, SDESC, SCNT, SIDX, SHI = 42, 43, 44, 45, 46, 47, 48, 49


def dpp(lane, ns):
    ctl = f"row_newbcast:{lane}" if ns <= 2 else f"quad_perm:[{lane},{lane},{lane},{lane}]"
    return f"{ctl} row_mask:0xf bank_mask:0xf"


def address_phase(e, vb, ns):
    L = []
    if ns <= 2:
        for u in range(UNITS):
            v = vb + 4 * u
            L += [f"v_xor_b32_dpp v{v}, v{e}, v31 {dpp(UNITS + u, ns)}",
                  f"ds_read_b128 v[{v}:{v + 3}], v{v}"]
    else:
        for u in range(2):
            v = vb + 16 * u
            L.append(f"v_xor_b32_dpp v{v}, v{e}, v31 {dpp(2 * u + 1, ns)}")
            for i in (1, 2, 3):             # quarters i ^ (g % 4): offsets 64, 128, 192 flipped
                L.append(f"v_xor_b32 v{v + 4 * i}, v{QREG + i - 1}, v{v}")
            for i in range(4):
                L.append(f"ds_read_b128 v[{v + 4 * i}:{v + 4 * i + 3}], v{v + 4 * i}")
    return L


def fmas(e, vb, ns, last=False):
    """The FMAs of a block whose 8 reads are the oldest in flight, 8 more behind them (or
    none: last)."""
    L = ["s_waitcnt lgkmcnt(0)"] if last else []
    if ns <= 2:
        if not last:
            L.append(f"s_waitcnt lgkmcnt({UNITS})")
        for u in range(UNITS):
            for k in range(4):
                L.append(f"v_fmac_f32_dpp v{ACC + 4 * (u % ns) + k}, v{e}, v{vb + 4 * u + k} {dpp(u, ns)}")
        return L
    for u in range(2):
        L.append(f"v_mov_b32_dpp v{WREG[u]}, v{e} {dpp(2 * u, ns)}")
    for u in range(2):
        acc = ACC + 16 * (u if ns == 8 else 0)
        for i in range(4):
            if not last:
                # (16 or 17 LDS instructions are in flight before the first wait: a 4-bit counter
                # at its end stands for 15 or more, so no wait is on 15)
                L.append(f"s_waitcnt lgkmcnt({min(14, 15 - (4 * u + i))})")
            for k in range(4):
                L.append(f"v_fmac_f32 v{acc + 4 * i + k}, v{WREG[u]}, v{vb + 16 * u + 4 * i + k}")
    return L


def lane0_write(addr, vdata):
    return ["s_mov_b64 exec, 1", f"ds_write_b32 {addr}, {vdata}", "s_mov_b64 exec, -1"]


def quarters(ns):
    return [] if ns <= 2 else [f"v_mov_b32 v{QREG + i}, {hex(64 * (i + 1))}" for i in range(3)]


def sync(tag, ns):
    """The sync point of the descriptor in SDESC: publish c_lo, wait for c_hi.  LDS
    executes a wave's instructions in order, so the reads issued before the progress word
    is written are done with their slots when a producer sees it.  Priority: raised at a
    sync point, dropped while polling (a wave that waits is ahead of its workgroup)."""
    L = ["s_setprio 1",
         f"s_bfe_u32 s{STMP}, s{SDESC}, {hex((HISHIFT - LOSHIFT) << 16 | LOSHIFT)}",
         f"s_add_u32 s{STMP}, s{STMP}, %[cbase]",
         f"v_mov_b32 v30, s{STMP}"]
    L += lane0_write("%[pa]", "v30")
    L += [f"s_lshr_b32 s{SHI}, s{SDESC}, {HISHIFT}",
          f".L%=_poll{tag}:",
          f"s_cmp_lt_u32 s{SHI}, s{SREADY}",
          f"s_cbranch_scc1 .L%=_ready{tag}",
          f"s_cmp_eq_u32 s{SPOLL}, 0",
          f"s_cbranch_scc1 .L%=_ready{tag}",
          f"s_sub_u32 s{SPOLL}, s{SPOLL}, 1",
          "s_setprio 0",
          "ds_read_b128 v[24:27], %[ra]",
          "s_waitcnt lgkmcnt(0)",
          # straight from the LDS result to SGPRs (a VALU write of a VGPR followed at
          # once by v_readfirstlane of it reads the old value)
          f"v_readfirstlane_b32 s{SREADY}, v24",
          f"v_readfirstlane_b32 s{SREADY1}, v25",
          f"s_min_u32 s{SREADY}, s{SREADY}, s{SREADY1}",
          f"v_readfirstlane_b32 s{SREADY1}, v26",
          f"s_min_u32 s{SREADY}, s{SREADY}, s{SREADY1}",
          f"v_readfirstlane_b32 s{SREADY1}, v27",
          f"s_min_u32 s{SREADY}, s{SREADY}, s{SREADY1}"] + quarters(ns) + [
          f"s_sub_u32 s{SREADY}, s{SREADY}, %[cbase]",   # chunks of this item landed
          f"s_max_i32 s{SREADY}, s{SREADY}, 0",
          f"s_cmp_lt_u32 s{SHI}, s{SREADY}",
          f"s_cbranch_scc1 .L%=_ready{tag}",
          "s_sleep 1",
          f"s_branch .L%=_poll{tag}",
          f".L%=_ready{tag}:"]
    return L


def consumer(ns):
    L = ["v_mov_b32 v28, %[l4]",
         "v_mov_b32 v31, %[vl]",
         f"s_mov_b64 s[{PTR}:{PTR + 1}], %[sp]",
         f"s_mov_b64 s[{DPTR}:{DPTR + 1}], %[dp]",
         f"s_mov_b32 s{SREADY}, 0",
         f"{'s_mov_b32' if ns == 8 else 'v_readfirstlane_b32'} s{SPOLL}, %[budget]",
         f"s_mov_b32 s{SIDX}, 0",
         f"global_load_dword v29, v28, s[{DPTR}:{DPTR + 1}]"]
    for e in range(NE):
        L.append(f"global_load_dword v{EREG + e}, v28, s[{PTR}:{PTR + 1}] offset:{256 * e}")
    L += [f"s_add_u32 s{PTR}, s{PTR}, {256 * NE}",
          f"s_addc_u32 s{PTR + 1}, s{PTR + 1}, 0",
          f"s_waitcnt vmcnt({NE})",
          f"v_readlane_b32 s{SDESC}, v29, s{SIDX}",
          f"s_and_b32 s{SCNT}, s{SDESC}, {hex(NMASK)}",
          f"s_sub_u32 s{SCNT}, s{SCNT}, 1"]
    L += quarters(ns) + sync("e", ns)
    L.append(f"s_waitcnt vmcnt({NE - 1})")
    L += address_phase(EREG, VB[0], ns)
    for i in range(NE):
        e, en = EREG + i, EREG + (i + 1) % NE
        b, bn = VB[i % 2], VB[(i + 1) % 2]
        if i == 0:
            L.append(".p2align 6")   # (off a cache line the loop ran up to 1.5 % slower)
        L += [f".L%=_iter{i}:",
              f"s_sub_u32 s{SCNT}, s{SCNT}, 1",
              f"s_cbranch_scc1 .L%=_sync{i}",
              f".L%=_ret{i}:",
              f"s_waitcnt vmcnt({NE - 2})"]
        L += address_phase(en, bn, ns)
        L += fmas(e, b, ns)
        L += [f"global_load_dword v{e}, v28, s[{PTR}:{PTR + 1}]",
              f"s_add_u32 s{PTR}, s{PTR}, 256",
              f"s_addc_u32 s{PTR + 1}, s{PTR + 1}, 0"]
    L.append("s_branch .L%=_iter0")
    for i in range(NE):
        L += [f".L%=_sync{i}:",
              f"s_add_u32 s{SIDX}, s{SIDX}, 1",
              f".L%=_desc{i}:",
              f"v_readlane_b32 s{SDESC}, v29, s{SIDX}",
              f"s_and_b32 s{SCNT}, s{SDESC}, {hex(NMASK)}",
              f"s_cbranch_scc0 .L%=_zero{i}",
              f"s_sub_u32 s{SCNT}, s{SCNT}, 1"]
        L += sync(i, ns)
        L += [f"s_branch .L%=_ret{i}",
              f".L%=_reload{i}:",              # the next 64 descriptors
              f"s_mov_b32 s{SIDX}, 0",
              f"s_add_u32 s{DPTR}, s{DPTR}, 256",
              f"s_addc_u32 s{DPTR + 1}, s{DPTR + 1}, 0",
              f"global_load_dword v29, v28, s[{DPTR}:{DPTR + 1}]",
              "s_waitcnt vmcnt(0)",
              f"s_branch .L%=_desc{i}",
              f".L%=_zero{i}:",
              f"s_cmp_lg_u32 s{SDESC}, 0",
              f"s_cbranch_scc1 .L%=_reload{i}"]
        L += fmas(EREG + i, VB[i % 2], ns, last=True)
        L.append("s_branch .L%=_finish")
    L += [".L%=_finish:",
          f"s_cmp_eq_u32 s{SPOLL}, 0", "s_cbranch_scc1 .L%=_poison",
          "ds_read_b32 v30, %[ov]", "s_waitcnt lgkmcnt(0)",
          f"v_readfirstlane_b32 s{STMP}, v30",
          f"s_cmp_eq_u32 s{STMP}, 0", "s_cbranch_scc1 .L%=_clean",
          ".L%=_poison:"]
    per = 4 if ns <= 2 else 16                      # accumulators per set
    sets = ns if ns <= 2 else ns // 4
    L += [f"v_mov_b32 v{ACC + x}, {hex(POISON)}" for x in range(per * sets)]
    L += [".L%=_clean:", f"{'s' if ns == 8 else 'v'}_mov_b32 %[budget], s{SPOLL}", "v_mov_b32 v30, %[next]"]
    L += lane0_write("%[pa]", "v30")
    L.append("s_waitcnt vmcnt(0) lgkmcnt(0)")
    body = "\n".join('      "' + x + '\\n\\t"' for x in L)
    accs = ", ".join(f'"+{{v[{ACC + per * q}:{ACC + per * (q + 1) - 1}]}}"(acc[{q}])' for q in range(sets))
    regs = [f"s{x}" for x in range(PTR, SHI + 1)] + [f"v{x}" for x in range(EREG, ACC)]
    clob = ", ".join(f'"{r}"' for r in regs + ["scc", "memory"])
    return f"""// Consumer, {4 * ns} rows per wave
__device__ __forceinline__ void consume_quads{ns}(group_acc_t<{per}> (&acc)[{sets}], QuadConsumer& a) {{
  uint32_t budget = {"__builtin_amdgcn_readfirstlane(a.poll_budget)" if ns == 8 else "a.poll_budget"};
  asm volatile(
{body}
      : {accs}, [budget] "+{'s' if ns == 8 else 'v'}"(budget)
      : [sp] "s"(a.stream), [dp] "s"(a.descs), [vl] "v"(a.vlane), [l4] "v"(a.lane4),
        [pa] "v"(a.prog_addr), [ra] "v"(a.ready_addr), [ov] "v"(a.overrun_addr),
        [cbase] "s"(a.chunk_base), [next] "s"(a.next_progress)
      : {clob});
  a.poll_budget = budget;
}}
"""


def generate() -> str:
    parts = ["// Generated by gen_quad_asm.py -- do not edit by hand.",
             "#pragma once", "",
             "// blocks the stream must carry past its last program (the loads run ahead)",
             f"constexpr int kQuadAsmTailBlocks = {NE + 1};",
             f"constexpr int kQuadAsmUnits = {UNITS}, kQuadAsmAccBase = {ACC};",
             f"constexpr int kQuadAsmLoShift = {LOSHIFT}, kQuadAsmHiShift = {HISHIFT};",
             f"constexpr uint32_t kQuadAsmCountMask = {hex(NMASK)}u, kQuadAsmPoison = {hex(POISON)}u;", ""]
    parts += [consumer(ns) for ns in NSETS]
    return "\n".join(parts)


def main(check: bool = False) -> int:
    text = generate()
    if check:
        return 0 if os.path.exists(OUT) and open(OUT).read() == text else 1
    with open(OUT, "w") as f:
        f.write(text)
    return 0


if __name__ == "__main__":
    sys.exit(main(check="--check" in sys.argv))
