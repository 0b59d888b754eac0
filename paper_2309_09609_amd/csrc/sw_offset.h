// 16-bit cells on anti-diagonal offsets: the local sweep's fast form.
//
// Included by sw_kernels.hip inside namespace sw, after the buffer access
// helpers, PassIO and Res.
//
// Cells store H, E and F plus an offset that grows by Ge from row to row of a
// lane and from step to step, phi(r, tau) = Go + Ge (r + tau) (tau counts steps
// from 1 and falls back by K every K steps, when everything held is lowered by
// Ge K).  On such cells a gap extends for free in both directions, and E and F
// open from the same value G = H - (Go - Ge):
//   hd = G(r-1, j-1) + (SM + Go + Ge)   the profile holds SM + Go + Ge, a byte
//   H  = maximum3(hd, E, F)
//   G  = H - (Go - Ge)                  kept instead of H
//   E' = maximum3(E, G, floor)          floor = phi of the next step: true 0
//   F' = max(F, G)
//   S  = maximum3(S, G(r, j), G(r+1, j-1))   two cells of one anti-diagonal
//                                       carry one offset; one S per two rows
// With Go >= Go - Ge every value stays non-negative without saturating
// arithmetic, so plain integer additions serve: one v_lshl_add_u64 forms the
// diagonal sums of two rows (four cells), and another raises two S words to
// the next step's offset.  Per row of two cells that is 5.25 instructions and,
// with two subjects per lane, one permute, against 7.5 and one for the plain
// biased form; the substitution bytes of 16 rows are one 16-byte LDS read per
// subject instead of two (and the 16-byte slots of 25 residues spread over all
// banks).
//
// What bounds it: VALU issue, 7.3 instructions per row of two cells over a whole
// 16-row step with two subjects per lane (9.5 in the plain form).  Measured
// against the plain form: 570,000 subjects, a query of 1,003 residues 27.3 ->
// 22.6 ms, of 5,478 149.4 -> 122.6 ms; 16 queries x 40,000 subjects, two queries
// per lane, 105.3 -> 82.2 ms; two queries of 330 - 361 x 200,000 10.8 -> 8.4 ms.
// (v_lshl_add_u64 issues at the rate of a 32-bit addition: 1.85 ns per wave and
// SIMD, as the packed maxima do.)
//
// Range: H <= 0x7BFF - phi is exact, as in the plain form (values below 0x7C00
// order like half floats; 0x7C00 and above are infinity or NaN and stay in S,
// whose own NaN v_pk_maximum3_f16 keeps, as the first operand).  The offsets
// cost Go + Ge (K + 17) of the range; the host recomputes pairs from there on
// (SweepArgs::sat).
//
// End-to-end modes (global, semi-global; Ge <= Go) run on the same cells without
// the floor: E' = max(E, G), and instead of S every G folds into a running
// minimum and maximum that tell whether all values stayed in the exact range.
// Values carry ec.bias instead of Go, just above the lowest value a pair can
// reach.  Global cells hold H + Ge j and so on (gap runs along the subject cost
// the offset's growth, and the border of row 0 is a constant), which is the
// same recurrence with no term in tau and nothing to lower.  5.5 instructions
// per row of two cells and a permute, against 8 and one for plain cells.  The
// last row's cells are read off once per step, only by the wave that holds them
// and in the columns that count.  Measured against the plain cells, with the
// longest pairs on a workgroup each (below): global, 405 residues x 570,000
// subjects, 17.5 -> 10.4 ms; semi-global, 331 x 100,000, 10.9 -> 2.15 ms.
//
// The rows' G live in fixed registers v64.. (row r's in v65 + r, the value
// above the block in v64) because v_lshl_add_u64 reads them in pairs and the
// rest one by one, which asm operands cannot express; so do S (v82..) and the
// block's temporaries (v90..v96).
//
// Schedule: no instruction reads the result of the packed (VOP3P) instruction
// just before it (a wait state the compiler cannot insert inside the block),
// and no DPP reads a register written by the two instructions before it.

struct CellOff : CellI16 {};

// What a launch's offset cells need, all packed twice into 32 bits.
struct OffCtx {
    uint32_t ge, goe;      // Ge, Go - Ge
    uint32_t go;           // Go
    int K;                 // steps between two renormalisations, a multiple of 4
};

#define SWO_P0 "v64"
#define SWO_P1 "v65"
#define SWO_P2 "v66"
#define SWO_P3 "v67"
#define SWO_P4 "v68"
#define SWO_P5 "v69"
#define SWO_P6 "v70"
#define SWO_P7 "v71"
#define SWO_P8 "v72"
#define SWO_P9 "v73"
#define SWO_P10 "v74"
#define SWO_P11 "v75"
#define SWO_P12 "v76"
#define SWO_P13 "v77"
#define SWO_P14 "v78"
#define SWO_P15 "v79"
#define SWO_P16 "v80"
#define SWO_PP0 "v[64:65]"
#define SWO_PP2 "v[66:67]"
#define SWO_PP4 "v[68:69]"
#define SWO_PP6 "v[70:71]"
#define SWO_PP8 "v[72:73]"
#define SWO_PP10 "v[74:75]"
#define SWO_PP12 "v[76:77]"
#define SWO_PP14 "v[78:79]"
#define SWO_S0 "v82"
#define SWO_S1 "v83"
#define SWO_S2 "v84"
#define SWO_S3 "v85"
#define SWO_S4 "v86"
#define SWO_S5 "v87"
#define SWO_S6 "v88"
#define SWO_S7 "v89"
#define SWO_SS0 "v[82:83]"
#define SWO_SS1 "v[84:85]"
#define SWO_SS2 "v[86:87]"
#define SWO_SS3 "v[88:89]"
// diagonal sums of a row pair, alternating between two register pairs
#define SWO_DA "v[92:93]"
#define SWO_DA0 "v92"
#define SWO_DA1 "v93"
#define SWO_DB "v[94:95]"
#define SWO_DB0 "v94"
#define SWO_DB1 "v95"

#define SWO_M(d, r) "v_pk_maximum3_f16 v96, " d ", %[e" #r "], %[f]\n"
#define SWO_G(p) "v_subrev_u32 " p ", %[goe], v96\n"
#define SWO_F(p) "v_pk_max_i16 %[f], %[f], " p "\n"
#define SWO_E(r, p) "v_pk_maximum3_f16 %[e" #r "], %[e" #r "], " p ", %[k" #r "]\n"
#define SWO_S(s, p, q) "v_pk_maximum3_f16 " s ", " s ", " p ", " q "\n"
#define SWO_SA(ss) "v_lshl_add_u64 " ss ", %[ge64], 0, " ss "\n"
// subject pairs: bytes q of a[w] and b[w], zero extended into the two halves
#define SWO_PERM(t, w, q) "v_perm_b32 " t ", %[b" #w "], %[a" #w "], %[q" #q "]\n"
#define SWO_HD(d, pp) "v_lshl_add_u64 " d ", " pp ", 0, v[90:91]\n"
// query pairs: w<k> holds the substitution pairs of rows 2k and 2k + 1
#define SWO_HDW(d, pp, k) "v_lshl_add_u64 " d ", " pp ", 0, %[w" #k "]\n"

// Rows r0, r1 (= r0 + 1) with their diagonal sums in d0, d1: G to p1, p2, where p2 and p3 hold the rows
// r1 and r1 + 1 of the previous column until then; the next pair's sums go to nd.  rp = the row before r0
// (its E update was left over; pp = its G).
#define SWO_BLK(d0, d1, nd, r0, r1, p1, p2, npp, s, w, qa, qb, EPREV)                                         \
    SWO_M(d0, r0) SWO_PERM("v90", w, qa) EPREV SWO_G(p1) SWO_F(p1) SWO_PERM("v91", w, qb) SWO_M(d1, r1)       \
    SWO_HD(nd, npp) SWO_S(s, p1, p2) SWO_G(p2) SWO_F(p2) SWO_E(r0, p1)
#define SWO_BLKW(d0, d1, nd, r0, r1, p1, p2, npp, s, w, EPREV)                                                \
    SWO_M(d0, r0) EPREV SWO_G(p1) SWO_F(p1) SWO_HDW(nd, npp, w) SWO_M(d1, r1)                                 \
    SWO_S(s, p1, p2) SWO_G(p2) SWO_F(p2) SWO_E(r0, p1)
// the last two rows: nothing to prepare, and F is followed by an instruction that leaves it alone
#define SWO_LAST(d0, d1, r0, r1, p1, p2, s, EPREV)                                                            \
    SWO_M(d0, r0) EPREV SWO_G(p1) SWO_F(p1) SWO_E(r0, p1) SWO_M(d1, r1) SWO_S(s, p1, p2) SWO_G(p2) SWO_F(p2)  \
    SWO_E(r1, p2)

// End-to-end modes: no floor, the range folds of a row pair behind its second F.  (E and G are plain integers: a
// half that fell below 0 reads 0xFF.., a NaN pattern, and stays in the folds.)
#define SWO_E0(r, p) "v_pk_max_i16 %[e" #r "], %[e" #r "], " p "\n"
#define SWO_FOLD(p, q) "v_pk_maximum3_f16 %[hi], %[hi], " p ", " q "\n" "v_pk_minimum3_f16 %[lo], %[lo], " p ", " q "\n"
#define SWO_MBLK(d0, d1, nd, r0, r1, p1, p2, npp, w, qa, qb, EPREV)                                           \
    SWO_M(d0, r0) SWO_PERM("v90", w, qa) EPREV SWO_G(p1) SWO_F(p1) SWO_PERM("v91", w, qb) SWO_M(d1, r1)       \
    SWO_HD(nd, npp) SWO_G(p2) SWO_F(p2) SWO_FOLD(p1, p2) SWO_E0(r0, p1)
#define SWO_MLAST(d0, d1, r0, r1, p1, p2, EPREV)                                                              \
    SWO_M(d0, r0) EPREV SWO_G(p1) SWO_F(p1) SWO_E0(r0, p1) SWO_M(d1, r1) "s_nop 0\n" SWO_G(p2) SWO_F(p2)      \
    SWO_FOLD(p1, p2) SWO_E0(r1, p2)

// What comes from above: a cooperating lane takes lane b-1's bottom row (its G and F of one step ago) and
// drops the rows' offset Ge (R - 1); the first lane of a group takes the boundary words, raised by as much.
#define SWO_TOP_COOP(pr)                                                                                      \
    "v_cndmask_b32_dpp %[f], %[f], %[bf], vcc wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n"           \
    "v_cndmask_b32_dpp v64, " pr ", %[bg], vcc wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n"          \
    "v_subrev_u32 %[f], %[cr], %[f]\n" "v_subrev_u32 v64, %[cr], v64\n"
#define SWO_TOP_ALONE "v_mov_b32 %[f], %[bf]\n" "v_mov_b32 v64, %[bg]\n"

#define SWO_PRE "s_mov_b64 vcc, %[first]\n" SWO_PERM("v90", 0, 0) SWO_PERM("v91", 0, 1)
#define SWO_ROWS4(TOP)                                                                                        \
    SWO_PRE SWO_SA(SWO_SS0) SWO_HD(SWO_DA, SWO_PP0) TOP                                                       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, SWO_S0, 0, 2, 3, "")                     \
    SWO_LAST(SWO_DB0, SWO_DB1, 2, 3, SWO_P3, SWO_P4, SWO_S1, SWO_E(1, SWO_P2))
#define SWO_ROWS8(TOP)                                                                                        \
    SWO_PRE SWO_SA(SWO_SS0) SWO_SA(SWO_SS1) SWO_HD(SWO_DA, SWO_PP0) TOP                                       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, SWO_S0, 0, 2, 3, "")                     \
    SWO_BLK(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, SWO_S1, 1, 0, 1, SWO_E(1, SWO_P2))       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, SWO_S2, 1, 2, 3, SWO_E(3, SWO_P4))       \
    SWO_LAST(SWO_DB0, SWO_DB1, 6, 7, SWO_P7, SWO_P8, SWO_S3, SWO_E(5, SWO_P6))
#define SWO_ROWS12(TOP)                                                                                       \
    SWO_PRE SWO_SA(SWO_SS0) SWO_SA(SWO_SS1) SWO_HD(SWO_DA, SWO_PP0) TOP SWO_SA(SWO_SS2)                       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, SWO_S0, 0, 2, 3, "")                     \
    SWO_BLK(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, SWO_S1, 1, 0, 1, SWO_E(1, SWO_P2))       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, SWO_S2, 1, 2, 3, SWO_E(3, SWO_P4))       \
    SWO_BLK(SWO_DB0, SWO_DB1, SWO_DA, 6, 7, SWO_P7, SWO_P8, SWO_PP8, SWO_S3, 2, 0, 1, SWO_E(5, SWO_P6))       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 8, 9, SWO_P9, SWO_P10, SWO_PP10, SWO_S4, 2, 2, 3, SWO_E(7, SWO_P8))     \
    SWO_LAST(SWO_DB0, SWO_DB1, 10, 11, SWO_P11, SWO_P12, SWO_S5, SWO_E(9, SWO_P10))
#define SWO_ROWS16(TOP)                                                                                       \
    SWO_PRE SWO_SA(SWO_SS0) SWO_SA(SWO_SS1) SWO_HD(SWO_DA, SWO_PP0) TOP SWO_SA(SWO_SS2) SWO_SA(SWO_SS3)       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, SWO_S0, 0, 2, 3, "")                     \
    SWO_BLK(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, SWO_S1, 1, 0, 1, SWO_E(1, SWO_P2))       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, SWO_S2, 1, 2, 3, SWO_E(3, SWO_P4))       \
    SWO_BLK(SWO_DB0, SWO_DB1, SWO_DA, 6, 7, SWO_P7, SWO_P8, SWO_PP8, SWO_S3, 2, 0, 1, SWO_E(5, SWO_P6))       \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 8, 9, SWO_P9, SWO_P10, SWO_PP10, SWO_S4, 2, 2, 3, SWO_E(7, SWO_P8))     \
    SWO_BLK(SWO_DB0, SWO_DB1, SWO_DA, 10, 11, SWO_P11, SWO_P12, SWO_PP12, SWO_S5, 3, 0, 1, SWO_E(9, SWO_P10)) \
    SWO_BLK(SWO_DA0, SWO_DA1, SWO_DB, 12, 13, SWO_P13, SWO_P14, SWO_PP14, SWO_S6, 3, 2, 3, SWO_E(11, SWO_P12)) \
    SWO_LAST(SWO_DB0, SWO_DB1, 14, 15, SWO_P15, SWO_P16, SWO_S7, SWO_E(13, SWO_P14))
// (end-to-end modes: a cooperating lane keeps its column-0 border until its first column)
#define SWO_MON "s_mov_b64 exec, %[act]\n"
#define SWO_MOFF "s_mov_b64 exec, -1\n"
#define SWO_MROWS4(TOP)                                                                                       \
    SWO_PRE SWO_HD(SWO_DA, SWO_PP0) TOP                                                                       \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, 0, 2, 3, "")                            \
    SWO_MLAST(SWO_DB0, SWO_DB1, 2, 3, SWO_P3, SWO_P4, SWO_E0(1, SWO_P2))
#define SWO_MROWS8(TOP)                                                                                       \
    SWO_PRE SWO_HD(SWO_DA, SWO_PP0) TOP                                                                       \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, 0, 2, 3, "")                            \
    SWO_MBLK(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, 1, 0, 1, SWO_E0(1, SWO_P2))             \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, 1, 2, 3, SWO_E0(3, SWO_P4))             \
    SWO_MLAST(SWO_DB0, SWO_DB1, 6, 7, SWO_P7, SWO_P8, SWO_E0(5, SWO_P6))
#define SWO_MROWS12(TOP)                                                                                      \
    SWO_PRE SWO_HD(SWO_DA, SWO_PP0) TOP                                                                       \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, 0, 2, 3, "")                            \
    SWO_MBLK(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, 1, 0, 1, SWO_E0(1, SWO_P2))             \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, 1, 2, 3, SWO_E0(3, SWO_P4))             \
    SWO_MBLK(SWO_DB0, SWO_DB1, SWO_DA, 6, 7, SWO_P7, SWO_P8, SWO_PP8, 2, 0, 1, SWO_E0(5, SWO_P6))             \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 8, 9, SWO_P9, SWO_P10, SWO_PP10, 2, 2, 3, SWO_E0(7, SWO_P8))           \
    SWO_MLAST(SWO_DB0, SWO_DB1, 10, 11, SWO_P11, SWO_P12, SWO_E0(9, SWO_P10))
#define SWO_MROWS16(TOP)                                                                                      \
    SWO_PRE SWO_HD(SWO_DA, SWO_PP0) TOP                                                                       \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, 0, 2, 3, "")                            \
    SWO_MBLK(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, 1, 0, 1, SWO_E0(1, SWO_P2))             \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, 1, 2, 3, SWO_E0(3, SWO_P4))             \
    SWO_MBLK(SWO_DB0, SWO_DB1, SWO_DA, 6, 7, SWO_P7, SWO_P8, SWO_PP8, 2, 0, 1, SWO_E0(5, SWO_P6))             \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 8, 9, SWO_P9, SWO_P10, SWO_PP10, 2, 2, 3, SWO_E0(7, SWO_P8))           \
    SWO_MBLK(SWO_DB0, SWO_DB1, SWO_DA, 10, 11, SWO_P11, SWO_P12, SWO_PP12, 3, 0, 1, SWO_E0(9, SWO_P10))       \
    SWO_MBLK(SWO_DA0, SWO_DA1, SWO_DB, 12, 13, SWO_P13, SWO_P14, SWO_PP14, 3, 2, 3, SWO_E0(11, SWO_P12))      \
    SWO_MLAST(SWO_DB0, SWO_DB1, 14, 15, SWO_P15, SWO_P16, SWO_E0(13, SWO_P14))
#define SWO_PREW "s_mov_b64 vcc, %[first]\n"
#define SWO_ROWS8W(TOP)                                                                                       \
    SWO_PREW SWO_SA(SWO_SS0) SWO_HDW(SWO_DA, SWO_PP0, 0) TOP                                                  \
    SWO_BLKW(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, SWO_S0, 1, SWO_SA(SWO_SS1))             \
    SWO_BLKW(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, SWO_S1, 2, SWO_E(1, SWO_P2))            \
    SWO_BLKW(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, SWO_S2, 3, SWO_E(3, SWO_P4))            \
    SWO_LAST(SWO_DB0, SWO_DB1, 6, 7, SWO_P7, SWO_P8, SWO_S3, SWO_E(5, SWO_P6))
#define SWO_ROWS16W(TOP)                                                                                      \
    SWO_PREW SWO_SA(SWO_SS0) SWO_SA(SWO_SS1) SWO_HDW(SWO_DA, SWO_PP0, 0) TOP SWO_SA(SWO_SS2)                  \
    SWO_BLKW(SWO_DA0, SWO_DA1, SWO_DB, 0, 1, SWO_P1, SWO_P2, SWO_PP2, SWO_S0, 1, SWO_SA(SWO_SS3))             \
    SWO_BLKW(SWO_DB0, SWO_DB1, SWO_DA, 2, 3, SWO_P3, SWO_P4, SWO_PP4, SWO_S1, 2, SWO_E(1, SWO_P2))            \
    SWO_BLKW(SWO_DA0, SWO_DA1, SWO_DB, 4, 5, SWO_P5, SWO_P6, SWO_PP6, SWO_S2, 3, SWO_E(3, SWO_P4))            \
    SWO_BLKW(SWO_DB0, SWO_DB1, SWO_DA, 6, 7, SWO_P7, SWO_P8, SWO_PP8, SWO_S3, 4, SWO_E(5, SWO_P6))            \
    SWO_BLKW(SWO_DA0, SWO_DA1, SWO_DB, 8, 9, SWO_P9, SWO_P10, SWO_PP10, SWO_S4, 5, SWO_E(7, SWO_P8))          \
    SWO_BLKW(SWO_DB0, SWO_DB1, SWO_DA, 10, 11, SWO_P11, SWO_P12, SWO_PP12, SWO_S5, 6, SWO_E(9, SWO_P10))      \
    SWO_BLKW(SWO_DA0, SWO_DA1, SWO_DB, 12, 13, SWO_P13, SWO_P14, SWO_PP14, SWO_S6, 7, SWO_E(11, SWO_P12))     \
    SWO_LAST(SWO_DB0, SWO_DB1, 14, 15, SWO_P15, SWO_P16, SWO_S7, SWO_E(13, SWO_P14))

#define SWO_OE(i) [e##i] "+v"(E[i])
#define SWO_E4 SWO_OE(0), SWO_OE(1), SWO_OE(2), SWO_OE(3)
#define SWO_E8 SWO_E4, SWO_OE(4), SWO_OE(5), SWO_OE(6), SWO_OE(7)
#define SWO_E12 SWO_E8, SWO_OE(8), SWO_OE(9), SWO_OE(10), SWO_OE(11)
#define SWO_E16 SWO_E8, SWO_OE(8), SWO_OE(9), SWO_OE(10), SWO_OE(11), SWO_OE(12), SWO_OE(13), SWO_OE(14), SWO_OE(15)
#define SWO_OP4 "+{v64}"(P[0]), "+{v65}"(P[1]), "+{v66}"(P[2]), "+{v67}"(P[3]), "+{v68}"(P[4])
#define SWO_OP8 SWO_OP4, "+{v69}"(P[5]), "+{v70}"(P[6]), "+{v71}"(P[7]), "+{v72}"(P[8])
#define SWO_OP12 SWO_OP8, "+{v73}"(P[9]), "+{v74}"(P[10]), "+{v75}"(P[11]), "+{v76}"(P[12])
#define SWO_OP16 SWO_OP12, "+{v77}"(P[13]), "+{v78}"(P[14]), "+{v79}"(P[15]), "+{v80}"(P[16])
#define SWO_OS4 "+{v82}"(S[0]), "+{v83}"(S[1])
#define SWO_OS8 SWO_OS4, "+{v84}"(S[2]), "+{v85}"(S[3])
#define SWO_OS12 SWO_OS8, "+{v86}"(S[4]), "+{v87}"(S[5])
#define SWO_OS16 SWO_OS8, "+{v86}"(S[4]), "+{v87}"(S[5]), "+{v88}"(S[6]), "+{v89}"(S[7])
#define SWO_K(i) [k##i] "s"(k[i])
#define SWO_K4 SWO_K(0), SWO_K(1), SWO_K(2), SWO_K(3)
#define SWO_K8 SWO_K4, SWO_K(4), SWO_K(5), SWO_K(6), SWO_K(7)
#define SWO_K12 SWO_K8, SWO_K(8), SWO_K(9), SWO_K(10), SWO_K(11)
#define SWO_K16 SWO_K8, SWO_K(8), SWO_K(9), SWO_K(10), SWO_K(11), SWO_K(12), SWO_K(13), SWO_K(14), SWO_K(15)
#define SWO_ABI(i) [a##i] "v"(w[i]), [b##i] "v"(w[R / 4 + i])
#define SWO_WI(i) [w##i] "v"(w64[i])
#define SWO_IN [bf] "v"(bf), [bg] "v"(bg), [goe] "s"(goe), [cr] "s"(cr), [ge64] "s"(ge64), [first] "s"(first)
#define SWO_INQ [q0] "s"(0x0c040c00u), [q1] "s"(0x0c050c01u), [q2] "s"(0x0c060c02u), [q3] "s"(0x0c070c03u)
#define SWO_CLOB "v90", "v91", "v92", "v93", "v94", "v95", "v96", "vcc"

// One column step of R rows, subject pairs: w holds R bytes of subject a's substitution scores, then of b's.
// P[0] = G above the block at the previous column, P[r + 1] = G of row r; F enters as lane b's F of the step
// before (handed to lane b + 1 here) and leaves as this step's.
template <int R, bool COOP>
__device__ __forceinline__ void rows_off_pair(uint32_t* P, uint32_t* E, uint32_t* S, uint32_t& F, uint32_t bg,
                                              uint32_t bf, const uint32_t* w, const uint32_t* k, uint32_t goe,
                                              uint32_t cr, uint64_t ge64, uint64_t first) {
    if constexpr (R == 16) {
        if constexpr (COOP)
            asm(SWO_ROWS16(SWO_TOP_COOP(SWO_P16)) : SWO_E16, [f] "+v"(F), SWO_OP16, SWO_OS16
                : SWO_IN, SWO_INQ, SWO_K16, SWO_ABI(0), SWO_ABI(1), SWO_ABI(2), SWO_ABI(3) : SWO_CLOB);
        else
            asm(SWO_ROWS16(SWO_TOP_ALONE) : SWO_E16, [f] "+v"(F), SWO_OP16, SWO_OS16
                : SWO_IN, SWO_INQ, SWO_K16, SWO_ABI(0), SWO_ABI(1), SWO_ABI(2), SWO_ABI(3) : SWO_CLOB);
    } else if constexpr (R == 12) {
        if constexpr (COOP)
            asm(SWO_ROWS12(SWO_TOP_COOP(SWO_P12)) : SWO_E12, [f] "+v"(F), SWO_OP12, SWO_OS12
                : SWO_IN, SWO_INQ, SWO_K12, SWO_ABI(0), SWO_ABI(1), SWO_ABI(2) : SWO_CLOB);
        else
            asm(SWO_ROWS12(SWO_TOP_ALONE) : SWO_E12, [f] "+v"(F), SWO_OP12, SWO_OS12
                : SWO_IN, SWO_INQ, SWO_K12, SWO_ABI(0), SWO_ABI(1), SWO_ABI(2) : SWO_CLOB);
    } else if constexpr (R == 8) {
        if constexpr (COOP)
            asm(SWO_ROWS8(SWO_TOP_COOP(SWO_P8)) : SWO_E8, [f] "+v"(F), SWO_OP8, SWO_OS8
                : SWO_IN, SWO_INQ, SWO_K8, SWO_ABI(0), SWO_ABI(1) : SWO_CLOB);
        else
            asm(SWO_ROWS8(SWO_TOP_ALONE) : SWO_E8, [f] "+v"(F), SWO_OP8, SWO_OS8
                : SWO_IN, SWO_INQ, SWO_K8, SWO_ABI(0), SWO_ABI(1) : SWO_CLOB);
    } else {
        static_assert(R == 4, "rows per lane must be 4, 8, 12 or 16");
        if constexpr (COOP)
            asm(SWO_ROWS4(SWO_TOP_COOP(SWO_P4)) : SWO_E4, [f] "+v"(F), SWO_OP4, SWO_OS4
                : SWO_IN, SWO_INQ, SWO_K4, SWO_ABI(0) : SWO_CLOB);
        else
            asm(SWO_ROWS4(SWO_TOP_ALONE) : SWO_E4, [f] "+v"(F), SWO_OP4, SWO_OS4
                : SWO_IN, SWO_INQ, SWO_K4, SWO_ABI(0) : SWO_CLOB);
    }
}

// End-to-end modes, subject pairs: lo and hi fold every G; lanes outside act keep everything.
template <int R, bool COOP>
__device__ __forceinline__ void rows_off_mode(uint32_t* P, uint32_t* E, uint32_t& lo, uint32_t& hi, uint32_t& F,
                                              uint32_t bg, uint32_t bf, const uint32_t* w, uint32_t goe, uint32_t cr,
                                              uint64_t first, uint64_t act) {
#define SWO_MASM(N, AB)                                                                                          \
    if constexpr (COOP)                                                                                               \
        asm(SWO_MON SWO_MROWS##N(SWO_TOP_COOP(SWO_P##N)) SWO_MOFF : SWO_E##N, [f] "+v"(F), SWO_OP##N, [lo] "+v"(lo), \
            [hi] "+v"(hi) : [bf] "v"(bf), [bg] "v"(bg), [goe] "s"(goe), [cr] "s"(cr), [first] "s"(first),            \
            [act] "s"(act), SWO_INQ, AB : SWO_CLOB);                                                                  \
    else                                                                                                              \
        asm(SWO_MROWS##N(SWO_TOP_ALONE) : SWO_E##N, [f] "+v"(F), SWO_OP##N, [lo] "+v"(lo), [hi] "+v"(hi)             \
            : [bf] "v"(bf), [bg] "v"(bg), [goe] "s"(goe), [cr] "s"(cr), [first] "s"(first), SWO_INQ, AB : SWO_CLOB)
#define SWO_AB4 SWO_ABI(0)
#define SWO_AB8 SWO_AB4, SWO_ABI(1)
#define SWO_AB12 SWO_AB8, SWO_ABI(2)
#define SWO_AB16 SWO_AB12, SWO_ABI(3)
    if constexpr (R == 16) { SWO_MASM(16, SWO_AB16); }
    else if constexpr (R == 12) { SWO_MASM(12, SWO_AB12); }
    else if constexpr (R == 8) { SWO_MASM(8, SWO_AB8); }
    else { static_assert(R == 4, "rows per lane must be 4, 8, 12 or 16"); SWO_MASM(4, SWO_AB4); }
}

// G of row r of the lane's block (r the same in every lane).  (Selects or an array index would send P to memory.)
#define SWO_IDX "s_set_gpr_idx_on %1, gpr_idx(SRC0)\n v_mov_b32 %0, v65\n s_set_gpr_idx_off"
#define SWO_IP4 "s"(r), "{v65}"(P[1]), "{v66}"(P[2]), "{v67}"(P[3]), "{v68}"(P[4])
#define SWO_IP8 SWO_IP4, "{v69}"(P[5]), "{v70}"(P[6]), "{v71}"(P[7]), "{v72}"(P[8])
#define SWO_IP12 SWO_IP8, "{v73}"(P[9]), "{v74}"(P[10]), "{v75}"(P[11]), "{v76}"(P[12])
#define SWO_IP16 SWO_IP12, "{v77}"(P[13]), "{v78}"(P[14]), "{v79}"(P[15]), "{v80}"(P[16])
template <int R>
__device__ __forceinline__ uint32_t row_g(const uint32_t* P, int r) {
    uint32_t g;
    if constexpr (R == 16) asm(SWO_IDX : "=v"(g) : SWO_IP16 : "m0");
    else if constexpr (R == 12) asm(SWO_IDX : "=v"(g) : SWO_IP12 : "m0");
    else if constexpr (R == 8) asm(SWO_IDX : "=v"(g) : SWO_IP8 : "m0");
    else asm(SWO_IDX : "=v"(g) : SWO_IP4 : "m0");
    return g;
}

// End-to-end modes: where a pass stands and what it takes from the query's last row.
struct EndOff {
    int row0;                  // 0-based first query row of this lane in this pass
    int m;
    int go, ge, bias;
    int na, nb;                // columns of the lane's two subjects (in a window: those before its end)
    int least, most;           // the smallest and largest of na and nb over the wave
    int rcap, bcap;            // row within the lane and lane within its group that hold the last row; rcap < 0: not in
                               // this wave or pass
    uint32_t lo = 0x7BFF7BFFu, hi = 0;   // range of every G
    uint32_t S = 0;            // semi-global: the largest G of the last row, global: the one at the last column
    __device__ int border(int k) const { return k <= 0 ? 0 : -(go + (k - 1) * ge); }   // Ge <= Go
};

// Column-0 borders of the R rows below row0 and their E at column 1; a lane that starts `late` steps in holds them at
// the offset of its first column (gt = what the offset grows by per step).
template <int R>
__device__ __forceinline__ void end_borders(const EndOff& ec, int gt, int late, uint32_t* P, uint32_t* E) {
#pragma unroll
    for (int r = 0; r <= R; ++r) {
        const uint32_t v = (uint32_t)(ec.border(min(ec.row0 + r, ec.m)) + ec.bias + ec.ge * r - ec.go + gt * late);
        P[r] = v | (v << 16);
        if (r < R) {
            const uint32_t e = (uint32_t)(ec.border(min(ec.row0 + r + 1, ec.m)) - ec.go + ec.bias + ec.ge * (r + 1) + gt * late);
            E[r] = e | (e << 16);
        }
    }
}

// What chunk c's steps take from the last row: 0 nothing, 1 (semi-global) every column of every lane, 2 by column.
template <int MODE>
__device__ __forceinline__ int end_takes(const EndOff& ec, int c) {
    const int col = 4 * c - ec.bcap;           // the column the lanes of the last row are at in the first step
    if (ec.rcap < 0 || col + 3 < (MODE == 1 ? max(ec.least, 1) - 1 : 0) || col >= ec.most) return 0;
    return MODE == 2 && col >= 0 && col + 3 < ec.least ? 1 : 2;
}

// The last row's cell of step t, offset `off` included in G (two halves alike).
template <int R, int MODE>
__device__ __forceinline__ void end_capture(EndOff& ec, int takes, const uint32_t* P, int t, uint32_t off) {
    asm volatile("" : "+s"(takes));           // (a scalar compare and branch per step, no masks kept)
    if (takes == 0) return;
    uint32_t g = row_g<R>(P, ec.rcap);
    const int col = t - ec.bcap;
    if constexpr (MODE == 1) {
        asm volatile("" : "+v"(g));
        if (col == ec.na - 1) ec.S = (ec.S & 0xffff0000u) | (g & 0xffffu);
        if (col == ec.nb - 1) ec.S = (ec.S & 0xffffu) | (g & 0xffff0000u);
    } else {
        g -= off;
        if (takes == 2) {                      // (a branch: few chunks of a pass take it)
            asm volatile("" : "+v"(g));
            g = col < 0 ? 0u : g & ((col < ec.na ? 0xffffu : 0u) | (col < ec.nb ? 0xffff0000u : 0u));
        }
        ec.S = bits<uint32_t>(__builtin_elementwise_max(bits<u2>(ec.S), bits<u2>(g)));
    }
}

// End-to-end modes on offset cells: the last row's cell that counts before any column (semi-global: column 0), a
// score from a captured G, and whether some G left the exact range.
template <int MODE>
__device__ __forceinline__ uint32_t end_start(const EndOff& ec, int r) {
    if (MODE == 1) return 0;
    return (uint32_t)(ec.border(ec.m) + ec.bias + ec.ge * r - (ec.go - ec.ge)) * 0x10001u;
}
template <int MODE>
__device__ __forceinline__ int end_score(const EndOff& ec, int g, int r, int n) {
    if (n == 0) return ec.border(ec.m);
    return g + ec.go - ec.ge - ec.bias - ec.ge * r - (MODE == 1 ? ec.ge * n : 0);
}
__device__ __forceinline__ bool end_outside(const EndOff& ec, int sat) {
    const u2 lo = bits<u2>(ec.lo), hi = bits<u2>(ec.hi);
    // (a NaN pattern, from either end, is above sat in hi)
    return lo.x < kOffLo || lo.y < kOffLo || (int)hi.x >= sat || (int)hi.y >= sat;
}

// Query pairs: w[r] = row r's substitution pair (both halves non-negative).
template <int R, bool COOP>
__device__ __forceinline__ void rows_off_packed(uint32_t* P, uint32_t* E, uint32_t* S, uint32_t& F, uint32_t bg,
                                                uint32_t bf, const uint32_t* w, const uint32_t* k, uint32_t goe,
                                                uint32_t cr, uint64_t ge64, uint64_t first) {
    uint64_t w64[R / 2];
#pragma unroll
    for (int i = 0; i < R / 2; ++i) w64[i] = ((uint64_t)w[2 * i + 1] << 32) | w[2 * i];
    if constexpr (R == 16) {
        if constexpr (COOP)
            asm(SWO_ROWS16W(SWO_TOP_COOP(SWO_P16)) : SWO_E16, [f] "+v"(F), SWO_OP16, SWO_OS16
                : SWO_IN, SWO_K16, SWO_WI(0), SWO_WI(1), SWO_WI(2), SWO_WI(3), SWO_WI(4), SWO_WI(5), SWO_WI(6),
                  SWO_WI(7) : SWO_CLOB);
        else
            asm(SWO_ROWS16W(SWO_TOP_ALONE) : SWO_E16, [f] "+v"(F), SWO_OP16, SWO_OS16
                : SWO_IN, SWO_K16, SWO_WI(0), SWO_WI(1), SWO_WI(2), SWO_WI(3), SWO_WI(4), SWO_WI(5), SWO_WI(6),
                  SWO_WI(7) : SWO_CLOB);
    } else {
        static_assert(R == 8, "query pairs run 8 or 16 rows per lane");
        if constexpr (COOP)
            asm(SWO_ROWS8W(SWO_TOP_COOP(SWO_P8)) : SWO_E8, [f] "+v"(F), SWO_OP8, SWO_OS8
                : SWO_IN, SWO_K8, SWO_WI(0), SWO_WI(1), SWO_WI(2), SWO_WI(3) : SWO_CLOB);
        else
            asm(SWO_ROWS8W(SWO_TOP_ALONE) : SWO_E8, [f] "+v"(F), SWO_OP8, SWO_OS8
                : SWO_IN, SWO_K8, SWO_WI(0), SWO_WI(1), SWO_WI(2), SWO_WI(3) : SWO_CLOB);
    }
}

// Substitution values of one step: subject pairs read R bytes of each subject (slice [residue][R bytes]),
// query pairs R dwords of their residue, four rows at a time (slice [row / 4][residue][4 dwords]: the
// 16-byte slots of one read's residues spread over all banks).
template <int R, bool PACKED>
__device__ __forceinline__ void fetch_off(const uint8_t* lrow, typename Res<PACKED>::V rr, int u, uint32_t* out) {
    if constexpr (PACKED) {
        const int d = (rr >> (8 * u)) & 0xff;
        const uint8_t* q = lrow + d * 16;
#pragma unroll
        for (int v = 0; v < R / 4; ++v) {
            const uint4 x = *reinterpret_cast<const uint4*>(q + v * kNRes * 16);
            out[4 * v] = x.x; out[4 * v + 1] = x.y; out[4 * v + 2] = x.z; out[4 * v + 3] = x.w;
        }
    } else {
        const uint8_t* qa = lrow + ((rr.x >> (8 * u)) & 0xff) * R;
        const uint8_t* qb = lrow + ((rr.y >> (8 * u)) & 0xff) * R;
        if constexpr (R == 16) {
            const uint4 x = *reinterpret_cast<const uint4*>(qa), y = *reinterpret_cast<const uint4*>(qb);
            out[0] = x.x; out[1] = x.y; out[2] = x.z; out[3] = x.w;
            out[4] = y.x; out[5] = y.y; out[6] = y.z; out[7] = y.w;
        } else if constexpr (R == 12) {
            const uint32_t *x = reinterpret_cast<const uint32_t*>(qa), *y = reinterpret_cast<const uint32_t*>(qb);
#pragma unroll
            for (int i = 0; i < 3; ++i) { out[i] = x[i]; out[3 + i] = y[i]; }
        } else if constexpr (R == 8) {
            const uint2 x = *reinterpret_cast<const uint2*>(qa), y = *reinterpret_cast<const uint2*>(qb);
            out[0] = x.x; out[1] = x.y; out[2] = y.x; out[3] = y.y;
        } else {
            out[0] = *reinterpret_cast<const uint32_t*>(qa);
            out[1] = *reinterpret_cast<const uint32_t*>(qb);
        }
    }
}

__device__ __forceinline__ uint64_t pair64(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }
// Four 16-bit sums in one instruction: no half of a wraps; the uniform x counts for both words.  (From C++ the
// compiler makes a 64-bit multiply-add of it.)
__device__ __forceinline__ uint64_t add_pairs(uint64_t a, uint32_t x) {
    uint64_t r;
    asm("v_lshl_add_u64 %0, %1, 0, %2" : "=v"(r) : "v"(a), "s"(pair64(x, x)));
    return r;
}
__device__ __forceinline__ uint32_t sgpr(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// One pass on offset cells: as sweep_pass, with the boundary words G and F free of offsets (the zero border
// of a first pass reads as zeros).  S receives the true scores of the lane's two matrices.
// IO = false: the query's only pass, with no boundary row to read or write (of a lone wave's step at 4 rows per lane
// that is one instruction in six).
template <int R, bool COOP, bool PACKED, bool IO = true, int MODE = 0>
__device__ __forceinline__ void sweep_pass_off(const PassIO& io, int ncols, int B, int b, const uint8_t* lrow,
                                               const OffCtx& o, u2& S, EndOff& ec) {
    using RV = typename Res<PACKED>::V;
    constexpr int NW = PACKED ? R : R / 2;                 // dwords of substitution values per step
    const int nsteps = ncols + B - 1;
    const int nloop = (nsteps + 3) >> 2;
    const uint32_t ge = sgpr(o.ge), goe = sgpr(o.goe), go = sgpr(o.go);
    const uint64_t ge64 = ((uint64_t)ge << 32) | ge;
    const uint64_t first = __ballot(b == 0);
    const uint32_t gt = MODE == 1 ? 0u : ge;               // growth of the offset per step
    const uint32_t cr = ge * R - gt;                       // no half of a product leaves 16 bits (host check)
    uint32_t P[R + 1], E[R], Sx[R / 2];
    uint32_t F = ge * R;                                   // what lane b-1 hands over before its first column
    uint32_t top0 = 0;                                     // the border of row 0 (G and F of the row above)
    if constexpr (MODE == 0) {
        // tau = 1 at the first step: G of column 0 carries Ge r, E of column 1 the floor Go + Ge (r + 1)
#pragma unroll
        for (int r = 0; r <= R; ++r) P[r] = ge * r;
#pragma unroll
        for (int r = 0; r < R; ++r) E[r] = go + ge * (r + 1);
#pragma unroll
        for (int i = 0; i < R / 2; ++i) Sx[i] = ge * (2 * i + 1);
    } else {
        end_borders<R>(ec, MODE == 1 ? 0 : ec.ge, COOP ? b : 0, P, E);
        if (io.first) top0 = (uint32_t)(ec.bias - ec.go - (MODE == 1 ? ec.go - ec.ge : 0)) * 0x10001u;
    }
    uint64_t act = first;                                  // lanes that have reached their first column
    int tau = 1;                                           // of the chunk's first step
    const int coff = COOP ? ((-b) >> 2) : 0;
    const int csh = COOP ? ((-b) & 3) : 0;
    auto res_at = [&](int c) { return Res<PACKED>::load(io.img, io.img_lane + (uint32_t)(c * kChunkBytes)); };
    auto resid = [&](RV lo, RV hi) { return COOP ? Res<PACKED>::align(hi, lo, csh) : lo; };
    RV c0 = res_at(coff), c1 = res_at(coff + 1), c2 = res_at(coff + 2);
    uint4 bw[2] = {};
    if constexpr (IO)
#pragma unroll
        for (int i = 0; i < 2; ++i) bw[i] = ld128(io.bnd, io.rd_lane + 16u * i);
    RV rr = resid(c0, c1);
    // subject pairs read their substitution bytes two steps ahead, query pairs (four times the words) one
    constexpr bool kLead2 = !PACKED;
    uint32_t cur[NW], nxt[NW];
    fetch_off<R, PACKED>(lrow, rr, 0, cur);
    if constexpr (kLead2) fetch_off<R, PACKED>(lrow, rr, 1, nxt);
    for (int c = 0; c < nloop; ++c) {
        const RV c3 = res_at(coff + c + 3);
        uint4 nw[2] = {};
        if constexpr (IO)
#pragma unroll
            for (int i = 0; i < 2; ++i) nw[i] = ld128(io.bnd, io.rd_lane + (uint32_t)(c + 1) * io.cstride + 16u * i);
        const RV rn = resid(c1, c2);
        const uint32_t get = gt * (uint32_t)tau;           // Ge tau of the chunk's first step
        uint32_t kk[R + 3];                                // floors of the next step, row r at step u: kk[r + u]
#pragma unroll
        for (int i = 0; i < R + 3; ++i) kk[i] = go + get + ge * (uint32_t)(i + 1);
        const uint32_t b0 = get + (COOP ? cr : 0u) + top0;
        const int takes = MODE != 0 ? end_takes<MODE>(ec, c) : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t nx2[NW];
            if constexpr (kLead2) {
                if (u < 2) fetch_off<R, PACKED>(lrow, rr, u + 2, nx2);
                else fetch_off<R, PACKED>(lrow, rn, u - 2, nx2);
            } else {
                if (u < 3) fetch_off<R, PACKED>(lrow, rr, u + 1, nxt);
                else fetch_off<R, PACKED>(lrow, rn, 0, nxt);
            }
            // the column's boundary words at this step's offset (no half leaves 16 bits)
            const uint4 v = bw[u >> 1];
            uint32_t bg = b0 + gt * u, bf = bg;
            if constexpr (IO) {
                const uint64_t top = add_pairs((u & 1) ? pair64(v.z, v.w) : pair64(v.x, v.y), b0 + gt * u);
                bg = (uint32_t)top;
                bf = (uint32_t)(top >> 32);
            }
            if constexpr (MODE != 0) {
                rows_off_mode<R, COOP>(P, E, ec.lo, ec.hi, F, bg, bf, cur, goe, cr, first, act);
                act = (act << 1) | first;
                end_capture<R, MODE>(ec, takes, P, 4 * c + u, get + gt * u);
            } else if constexpr (PACKED) rows_off_packed<R, COOP>(P, E, Sx, F, bg, bf, cur, kk + u, goe, cr, ge64, first);
            else rows_off_pair<R, COOP>(P, E, Sx, F, bg, bf, cur, kk + u, goe, cr, ge64, first);
            // the last lane of a lane group hands column j = t - (B - 1) to the next pass, without offset
            if constexpr (IO) {
                const int j = 4 * c + u - (B - 1);
                const uint32_t off = get + ge * (uint32_t)R + gt * u;
                st64(io.bnd, io.wr_lane + (uint32_t)((j >> 2) * (int)io.cstride + (j & 3) * 8), P[R] - off, F - off);
            }
#pragma unroll
            for (int r = 0; r < NW; ++r) {
                cur[r] = nxt[r];
                if constexpr (kLead2) nxt[r] = nx2[r];
            }
        }
        tau += 4;
        if (MODE != 1 && tau > o.K) {                      // lower everything by Ge K
            const uint32_t down = ge * (uint32_t)o.K;
#pragma unroll
            for (int r = 0; r <= R; ++r) P[r] -= down;
#pragma unroll
            for (int r = 0; r < R; ++r) E[r] -= down;
            if constexpr (MODE == 0)
#pragma unroll
                for (int i = 0; i < R / 2; ++i) Sx[i] -= down;
            F -= down;
            tau -= o.K;
        }
        c0 = c1;
        c1 = c2;
        c2 = c3;
        rr = rn;
#pragma unroll
        for (int i = 0; i < 2; ++i) bw[i] = nw[i];
    }
    if constexpr (MODE != 0) return;
    // S[i] stands at offset Ge (2i + 1 + tau) of the last step (tau - 1 now); the odd rows of the last column
    // were not folded yet (their own offset is Ge more).  Infinity and NaN patterns stay above every score.
    const uint32_t last = ge * (uint32_t)(tau - 1);
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
        const u2 x = __builtin_elementwise_sub_sat(bits<u2>(Sx[i]), bits<u2>(last + ge * (uint32_t)(2 * i + 1)));
        const u2 y = __builtin_elementwise_sub_sat(bits<u2>(P[2 * i + 2]), bits<u2>(last + ge * (uint32_t)(2 * i + 2)));
        S = __builtin_elementwise_max(S, __builtin_elementwise_max(x, y));
    }
}

// Rows [row0, row0 + B*R) of a query profile (int16, SM + Go + Ge on real residues) into LDS as bytes
// [b][residue][R].
template <int R>
__device__ __forceinline__ void load_slice_off(uint8_t* dst, const int16_t* prof, int mp, int row0, int lgB, int tid,
                                               int nthreads) {
    constexpr int U = (R % 8 == 0) ? 8 : 4;
    const int per_res = (R << lgB) / U;
    const int total = kNRes * per_res;
    for (int e = tid; e < total; e += nthreads) {
        const int d = e / per_res;
        const int rem = e - d * per_res;
        const int bb = rem / (R / U);
        const int ru = rem - bb * (R / U);
        const int16_t* src = prof + (int64_t)d * mp + row0 + rem * U;
        uint8_t* out = dst + (bb * kNRes + d) * R + ru * U;
        if constexpr (U == 8) {
            const uint4 v = *reinterpret_cast<const uint4*>(src);
            *reinterpret_cast<uint2*>(out) = make_uint2(__builtin_amdgcn_perm(v.y, v.x, 0x06040200u),
                                                        __builtin_amdgcn_perm(v.w, v.z, 0x06040200u));
        } else {
            const uint2 v = *reinterpret_cast<const uint2*>(src);
            *reinterpret_cast<uint32_t*>(out) = __builtin_amdgcn_perm(v.y, v.x, 0x06040200u);
        }
    }
}

// Rows [row0, row0 + B*R) of two query profiles interleaved into LDS as [b][row / 4][residue][4 dwords] (low
// half query a, high half query b).  Rows past a profile's stride read as padding (0).
template <int R>
__device__ __forceinline__ void load_slice_off_q2(uint32_t* dst, const int16_t* pa, int mpa, const int16_t* pb, int mpb,
                                                  int row0, int lgB, int tid, int nthreads) {
    const int per_res = (R << lgB) / 8;                 // 8-row units per residue
    const int total = kNRes * per_res;
    for (int e = tid; e < total; e += nthreads) {
        const int d = e / per_res;
        const int rem = e - d * per_res;
        const int row = row0 + rem * 8;
        const int bb = (rem * 8) / R;
        const int v0 = (rem * 8 - bb * R) / 4;
        uint4 va = make_uint4(0, 0, 0, 0), vb = va;
        if (row < mpa) va = *reinterpret_cast<const uint4*>(pa + (int64_t)d * mpa + row);
        if (row < mpb) vb = *reinterpret_cast<const uint4*>(pb + (int64_t)d * mpb + row);
        uint4 o0, o1;
        o0.x = __builtin_amdgcn_perm(vb.x, va.x, 0x05040100u); o0.y = __builtin_amdgcn_perm(vb.x, va.x, 0x07060302u);
        o0.z = __builtin_amdgcn_perm(vb.y, va.y, 0x05040100u); o0.w = __builtin_amdgcn_perm(vb.y, va.y, 0x07060302u);
        o1.x = __builtin_amdgcn_perm(vb.z, va.z, 0x05040100u); o1.y = __builtin_amdgcn_perm(vb.z, va.z, 0x07060302u);
        o1.z = __builtin_amdgcn_perm(vb.w, va.w, 0x05040100u); o1.w = __builtin_amdgcn_perm(vb.w, va.w, 0x07060302u);
        uint4* out = reinterpret_cast<uint4*>(dst) + ((bb * (R / 4) + v0) * kNRes + d);
        out[0] = o0;
        out[kNRes] = o1;
    }
}

// ------------------------------------------------------------ long subjects
// One subject pair on the four waves of a workgroup.  A subject much longer
// than a wave's share of the search is one serial chain of steps; here the
// chain is cut both ways:
//   * rows: wave w owns rows [64 R w, 64 R (w + 1)) of a pass and runs kChainLag
//     steps behind wave w - 1, whose bottom row reaches it through a ring of
//     columns in LDS (a workgroup barrier every kChainStage steps; a column is
//     written more than one stage before it is read, one chunk of read-ahead
//     included);
//   * columns: a query whose rows need one or two of the four waves lets the
//     others sweep further windows of the subject.  A window starts `span`
//     columns before its own ones: no local alignment with a positive score
//     covers more subject residues (QDesc::span), so each lies wholly in the
//     window that holds its end, and the score is the largest window's.  A pair
//     that would still outlast the search is split into parts, each with its
//     own windows, on a workgroup each; the last to end has the score.
// Every wave of a workgroup runs the same number of stages, and so of barriers,
// computed from the item before the first.
//
// A step of a lone wave takes less time than a load from memory is on its way for
// four of them, so global memory is read 64 chunks of residues (and 64 boundary
// columns) at a time, one of each lane, half a ring ahead, and passed on in LDS.
//
// Bound by the latency of a wave's step (about 60 instructions at 4 rows per
// lane, the fewest; more rows would need more LDS than the bulk units beside
// it leave).  The items run in the bulk launch itself, ahead of its units: a
// launch of their own on another stream shares a hardware queue with the bulk
// launch as soon as a process holds a few handles, and then runs before it
// instead of beside it.  One pair of 35,000 residues on one workgroup takes 1.3
// ms for a query of 200 residues (four windows), 2.4 ms for 331 and 4.4 ms for
// 1,024 (126 ns a step; global 161, semi-global 170, which also read the last
// row), in eight parts 0.35, 0.6 and 1.3 ms.  A query of 144 against 570,000
// subjects, the longest of 35,000 residues, went from 7.4 ms (a wave of its own
// for that pair) to 3.6 ms with it.
constexpr int kChainWaves = kWaves;
constexpr int kChainRows = 4;
constexpr int kChainStage = 16;              // steps between barriers (4 chunks)
constexpr int kChainLag = 96;                // steps between neighbouring waves: 64 lanes + 2 stages
constexpr int kChainRing = 256;              // columns of a ring
static_assert(kChainLag - 63 > kChainStage + 2 * kChunkCols, "a column is read after the barrier that follows its write");
static_assert(kChainLag % kChainStage == 0 && kChainRing > 2 * kChainLag, "ring and stages");
constexpr int kChainRingBytes = kChainRing * 8;
constexpr int kChainResBytes = 128 * 8;                    // residues of 128 chunks
constexpr int kChainIdle = kChainRingBytes + 64 * 8;       // where lanes that hand on nothing write
// LDS of a workgroup: the waves' slices, the ring that feeds each wave, their residues, the idle lanes' place, zeros
constexpr int kChainLds = kChainWaves * (64 * kNRes * kChainRows + kChainRingBytes + kChainResBytes) + kChainIdle + 32;

// The barrier between stages orders the rings in LDS only: what is on its way from or to global memory (residues
// and boundary words of later chunks) stays in flight, which a workgroup fence would wait for.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Wave w (of several on one window) for all its chunks of one pass; `stages` barriers pass whatever it does.
// STORE: the last wave's bottom row goes to the next pass through global memory.
template <int R, bool STORE, int MODE>
__device__ __forceinline__ void chain_pass(const PassIO& io, int ncols, int w, int stages, bool active, int b,
                                           const uint8_t* lrow, uint8_t* ring_in, uint8_t* out_lane, uint8_t* resq,
                                           const uint8_t* zeros, const OffCtx& o, u2& S, EndOff& ec) {
    using RV = uint2;
    constexpr int NW = R / 2;
    const int nloop = (ncols + 63 + 3) >> 2;
    const int first_stage = w * (kChainLag / kChainStage);
    const uint32_t ge = sgpr(o.ge), goe = sgpr(o.goe), go = sgpr(o.go);
    const uint64_t ge64 = ((uint64_t)ge << 32) | ge;
    const uint64_t first = 1;
    const uint32_t gt = MODE == 1 ? 0u : ge;
    const uint32_t cr = ge * R - gt;
    uint32_t P[R + 1], E[R], Sx[R / 2];
    uint32_t F = ge * R, top0 = 0;
    if constexpr (MODE == 0) {
#pragma unroll
        for (int r = 0; r <= R; ++r) P[r] = ge * r;
#pragma unroll
        for (int r = 0; r < R; ++r) E[r] = go + ge * (r + 1);
#pragma unroll
        for (int i = 0; i < R / 2; ++i) Sx[i] = ge * (2 * i + 1);
    } else {
        end_borders<R>(ec, MODE == 1 ? 0 : ec.ge, b, P, E);
        if (io.first && w == 0) top0 = (uint32_t)(ec.bias - ec.go - (MODE == 1 ? ec.go - ec.ge : 0)) * 0x10001u;
    }
    uint64_t act = first;
    int tau = 1;
    const int coff = (-b) >> 2, csh = (-b) & 3;
    // chunk b + 64 x of the residues, column b + 64 x of the boundary row (wave 0; zeros in the first pass)
    auto res_block = [&](int x) { return ld64(io.img, io.img_lane + (uint32_t)((64 * x + b) * kChunkBytes)); };
    // a residue byte becomes its slot's offset in the slice (at most 24 x 4)
    static_assert(R == 4, "residue x R fits a byte");
    auto stage_res = [&](int x, RV v) { *reinterpret_cast<RV*>(resq + ((64 * x + b) & 127) * 8) = RV{v.x * R, v.y * R}; };
    auto bnd_block = [&](int x) { return ld64(io.bnd, io.rd_lane + (uint32_t)(64 * x + b) * 8u); };
    auto res_at = [&](int c) { return *reinterpret_cast<const RV*>(resq + ((c + coff) & 127) * 8); };
    // the boundary words of chunk c
    // (past the subject the ring holds old columns: zeros instead)
    auto bound = [&](int c, uint4* v) {
        const uint4* q = reinterpret_cast<const uint4*>(4 * c < ncols ? ring_in + ((4 * c) & (kChainRing - 1)) * 8 : zeros);
        v[0] = q[0];
        v[1] = q[1];
    };
    // substitution bytes of column u of a chunk
    auto bytes = [&](RV v, int u, uint32_t* out) {
        out[0] = *reinterpret_cast<const uint32_t*>(lrow + ((v.x >> (8 * u)) & 0xff));
        out[1] = *reinterpret_cast<const uint32_t*>(lrow + ((v.y >> (8 * u)) & 0xff));
    };
    RV c0 = {}, c1 = {}, c2 = {}, rr = {}, res_next = {}, bnd_next = {};
    uint4 bw[2] = {};
    uint32_t cur[NW], nxt[NW];
    for (int i = 0; i < NW; ++i) cur[i] = nxt[i] = 0;
    for (int s = 0; s < stages; ++s) {
        const int ls = s - first_stage;
        if (active && ls >= 0 && ls * (kChainStage / 4) < nloop) {
            if (ls == 0) {
                const RV r0 = res_block(0);
                res_next = res_block(1);
                stage_res(1, RV{0, 0});                          // columns before the first
                stage_res(0, r0);
                if (w == 0) {
                    const RV b0 = bnd_block(0);
                    bnd_next = bnd_block(1);
                    *reinterpret_cast<RV*>(ring_in + b * 8) = b0;
                }
                c0 = res_at(0);
                c1 = res_at(1);
                c2 = res_at(2);
                bound(0, bw);
                rr = Res<false>::align(c1, c0, csh);
                bytes(rr, 0, cur);
                bytes(rr, 1, nxt);
            }
            const int c_end = min(nloop, (ls + 1) * (kChainStage / 4));
            for (int c = ls * (kChainStage / 4); c < c_end; ++c) {
                // half way through a block its successor goes to LDS and the next one is asked for
                if ((c & 63) == 32) {
                    const int x = (c >> 6) + 1;
                    stage_res(x, res_next);
                    res_next = res_block(x + 1);
                }
                if (w == 0 && (c & 15) == 8) {
                    const int x = (c >> 4) + 1;
                    *reinterpret_cast<RV*>(ring_in + ((64 * x + b) & (kChainRing - 1)) * 8) = bnd_next;
                    bnd_next = bnd_block(x + 1);
                }
                const RV c3 = res_at(c + 3);
                uint4 nw[2];
                bound(c + 1, nw);
                const RV rn = Res<false>::align(c2, c1, csh);
                const uint32_t get = gt * (uint32_t)tau;
                uint32_t kk[R + 3];
#pragma unroll
                for (int i = 0; i < R + 3; ++i) kk[i] = go + get + ge * (uint32_t)(i + 1);
                const uint32_t b0 = get + cr + top0;
                const int takes = MODE != 0 ? end_takes<MODE>(ec, c) : 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint32_t nx2[NW];
                    if (u < 2) bytes(rr, u + 2, nx2);
                    else bytes(rn, u - 2, nx2);
                    // G and F of the row above, raised to this step's offset (no half leaves 16 bits)
                    const uint4 v = bw[u >> 1];
                    const uint64_t top = add_pairs((u & 1) ? pair64(v.z, v.w) : pair64(v.x, v.y), b0 + gt * u);
                    const uint32_t bg = (uint32_t)top, bf = (uint32_t)(top >> 32);
                    if constexpr (MODE != 0) {
                        rows_off_mode<R, true>(P, E, ec.lo, ec.hi, F, bg, bf, cur, goe, cr, first, act);
                        act = (act << 1) | first;
                        end_capture<R, MODE>(ec, takes, P, 4 * c + u, get + gt * u);
                    } else
                        rows_off_pair<R, true>(P, E, Sx, F, bg, bf, cur, kk + u, goe, cr, ge64, first);
                    const int j = 4 * c + u - 63;
                    const uint32_t off = get + ge * (uint32_t)R + gt * u;
                    const uint2 down = make_uint2(P[R] - off, F - off);
                    *reinterpret_cast<uint2*>(out_lane + (j & (kChainRing - 1)) * 8) = down;
                    if constexpr (STORE)
                        st64(io.bnd, io.wr_lane + (uint32_t)((j >> 2) * (int)io.cstride + (j & 3) * 8), down.x, down.y);
#pragma unroll
                    for (int r = 0; r < NW; ++r) { cur[r] = nxt[r]; nxt[r] = nx2[r]; }
                }
                tau += 4;
                if (MODE != 1 && tau > o.K) {
                    const uint32_t down = ge * (uint32_t)o.K;
#pragma unroll
                    for (int r = 0; r <= R; ++r) P[r] -= down;
#pragma unroll
                    for (int r = 0; r < R; ++r) E[r] -= down;
                    if constexpr (MODE == 0)
#pragma unroll
                        for (int i = 0; i < R / 2; ++i) Sx[i] -= down;
                    F -= down;
                    tau -= o.K;
                }
                c0 = c1;
                c1 = c2;
                c2 = c3;
                rr = rn;
                bw[0] = nw[0];
                bw[1] = nw[1];
            }
        }
        stage_barrier();
    }
    if (!active || MODE != 0) return;
    const uint32_t last = ge * (uint32_t)(tau - 1);
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
        const u2 x = __builtin_elementwise_sub_sat(bits<u2>(Sx[i]), bits<u2>(last + ge * (uint32_t)(2 * i + 1)));
        const u2 y = __builtin_elementwise_sub_sat(bits<u2>(P[2 * i + 2]), bits<u2>(last + ge * (uint32_t)(2 * i + 2)));
        S = __builtin_elementwise_max(S, __builtin_elementwise_max(x, y));
    }
}
