// Term streaming with the points' coordinates in vector registers.
//
// A monomial is the product of the coordinates its factor list names, the
// same for every lane (a lane is a point).  From LDS each factor costs a
// 512-byte read per wave, and the four SIMDs of a CU share 128 bytes per
// clock: 16 clocks per factor and SIMD, four times what the multiplication
// itself takes.  Here the coordinates x_0 .. x_n (x_n = 1, the padding of
// short lists) sit in consecutive register pairs, and a factor is a
// multiplication whose first operand is named by the index register
// (s_set_gpr_idx_*).  A SIMD issues one scalar and one vector instruction
// every four clocks, so scalar work counts as much as the arithmetic: one
// 64-bit shift serves the factor bytes of two terms, and up to 55 variables a
// lane holds two points, which share every index.  (One index and one shift
// per multiplication: 9.3 clocks; one index: 4.4; one index for two
// multiplications: 2.2 and then 4.3 for the multiplications, measured with
// two waves on a SIMD.)
//
// The compiler has no way to keep an array of more than 16 doubles in
// registers that way, so the loop over a range of terms is one block of
// assembly: it reads the coordinates from the workgroup's tile and streams
// the terms in groups.  Scalar loads return in any order and can only be
// waited for all together, 1,100 clocks after the issue when the terms come
// from L2: factor bytes are read 32 terms ahead (16 beyond four factors), a
// register each, which that many terms' arithmetic hides, and coefficients
// take no scalar registers: lane l reads that of term l mod 16, and the
// multiply-add takes term k's from lane k of each row of 16 (row_newbcast).
// Every wait is within the block.  A term is ((x_a x_b) x_c) .., then a fused
// multiply-add with its coefficient, terms in order: the operations of the
// LDS form, to the bit.  Four products are interleaved.
//
// Registers named outright: the coordinates', from RE_BASE on, and s36-s99.
#pragma once

#include "kernels.h"

namespace polyhip {

// Two factor words' bytes (2 i for variable i) move down together.
#define RE_SHR(w) "s_lshr_b64 s[" w ":" w "+1], s[" w ":" w "+1], 8\n"
#define RE_MUL(t, x) "v_mul_f64 " t ", " x ", " t "\n"
#define RE_ONE(t, x) "v_mul_f64 " t ", " x ", 1.0\n"
#define RE_IDX(w) "s_set_gpr_idx_idx s[" w "]\n"
#define RE_ON(w) "s_set_gpr_idx_on s[" w "], gpr_idx(SRC0)\n"
#define RE_ADD(acc, c, t, k) "v_fmac_f64_dpp " acc ", " c ", " t " row_newbcast:re_k+" k " row_mask:0xf bank_mask:0xf\n"

// Four products: of four terms at one point (RE_*1), of two terms at two
// points (RE_*2).  X, Y: the first coordinate of the points; w: the symbol
// that holds the first term's word register.
#define RE_FIRST1(X, Y)                                                                       \
    RE_ON("re_w") RE_ONE("%[t0]", X) RE_IDX("re_w+1") RE_ONE("%[t1]", X)                       \
    RE_IDX("re_w+2") RE_ONE("%[t2]", X) RE_IDX("re_w+3") RE_ONE("%[t3]", X)
#define RE_SAME1(X, Y, w)                                                                     \
    RE_IDX(w) RE_MUL("%[t0]", X) RE_IDX(w "+1") RE_MUL("%[t1]", X)                             \
    RE_IDX(w "+2") RE_MUL("%[t2]", X) RE_IDX(w "+3") RE_MUL("%[t3]", X)
#define RE_NEXT1(X, Y, w) RE_SHR(w) RE_SHR(w "+2") RE_SAME1(X, Y, w)
#define RE_LAST1(c)                                                                           \
    "s_set_gpr_idx_off\n" RE_ADD("%[acc0]", c, "%[t0]", "0") RE_ADD("%[acc0]", c, "%[t1]", "1") \
    RE_ADD("%[acc0]", c, "%[t2]", "2") RE_ADD("%[acc0]", c, "%[t3]", "3")                      \
    ".set re_w, re_w+4\n.set re_u, re_u+4\n.set re_k, re_k+4\n"
#define RE_FIRST2(X, Y)                                                                       \
    RE_ON("re_w") RE_ONE("%[t0]", X) RE_ONE("%[t1]", Y) RE_IDX("re_w+1") RE_ONE("%[t2]", X) RE_ONE("%[t3]", Y)
#define RE_SAME2(X, Y, w)                                                                     \
    RE_IDX(w) RE_MUL("%[t0]", X) RE_MUL("%[t1]", Y) RE_IDX(w "+1") RE_MUL("%[t2]", X) RE_MUL("%[t3]", Y)
#define RE_NEXT2(X, Y, w) RE_SHR(w) RE_SAME2(X, Y, w)
#define RE_LAST2(c)                                                                           \
    "s_set_gpr_idx_off\n" RE_ADD("%[acc0]", c, "%[t0]", "0") RE_ADD("%[acc1]", c, "%[t1]", "0") \
    RE_ADD("%[acc0]", c, "%[t2]", "1") RE_ADD("%[acc1]", c, "%[t3]", "1")                      \
    ".set re_w, re_w+2\n.set re_u, re_u+2\n.set re_k, re_k+2\n"

// by number of factors
#define RE_LIST2(P, X, Y) RE_FIRST##P(X, Y) RE_NEXT##P(X, Y, "re_w")
#define RE_LIST3(P, X, Y) RE_LIST2(P, X, Y) RE_NEXT##P(X, Y, "re_w")
#define RE_LIST4(P, X, Y) RE_LIST3(P, X, Y) RE_NEXT##P(X, Y, "re_w")
#define RE_LIST5(P, X, Y) RE_LIST4(P, X, Y) RE_SAME##P(X, Y, "re_u")
#define RE_LIST6(P, X, Y) RE_LIST5(P, X, Y) RE_NEXT##P(X, Y, "re_u")
#define RE_LIST8(P, X, Y) RE_LIST6(P, X, Y) RE_NEXT##P(X, Y, "re_u") RE_NEXT##P(X, Y, "re_u")

// Sixteen terms in two octets (the block ends where none is left), then the
// load of the coefficients after the next sixteen; past the range a lane
// reads the range's last one again.
#define RE_OCTET(C, P, X, Y, c)                                                               \
    "s_sub_u32 %[q], %[q], 1\ns_cbranch_scc1 9f\n.rept " #P "*2\n" RE_LIST##C(P, X, Y) RE_LAST##P(c) ".endr\n"
#define RE_HALF(C, P, X, Y, c)                                                                \
    ".set re_k, 0\ns_waitcnt vmcnt(1)\n" RE_OCTET(C, P, X, Y, c) RE_OCTET(C, P, X, Y, c) RE_COEFS(c)
#define RE_COEFS(c) \
    "v_add_u32 %[vo], 0x80, %[vo]\nv_min_u32 %[vo], %[vo], %[vm]\nglobal_load_dwordx2 " c ", %[vo], %[cp]\n"

// A register set: 32 words, or the two words of 16 terms.  Its loads were
// issued one set earlier; those of the next are issued first, if it has terms.
#define RE_LOAD_SHORT(r) \
    "s_load_dwordx16 s[" #r ":" #r "+15], %[wp], %[wo]\ns_load_dwordx16 s[" #r "+16:" #r "+31], %[wp], %[wo2]\n"
#define RE_LOAD_LONG(r) \
    "s_load_dwordx16 s[" #r ":" #r "+15], %[wp], %[wo]\ns_load_dwordx16 s[" #r "+16:" #r "+31], %[up], %[wo]\n"
#define RE_SET_SHORT(C, P, X, Y, r, next, c)                                                   \
    "s_waitcnt lgkmcnt(0)\ns_cmp_le_u32 %[q], 4\ns_cbranch_scc1 2f\n"                            \
    "s_add_u32 %[wo], %[wo], 128\ns_add_u32 %[wo2], %[wo2], 128\n" RE_LOAD_SHORT(next)          \
    "2:\n.set re_w, " #r "\n" RE_HALF(C, P, X, Y, "%[c0]") RE_HALF(C, P, X, Y, "%[c1]")
#define RE_SET_LONG(C, P, X, Y, r, next, c)                                                    \
    "s_waitcnt lgkmcnt(0)\ns_cmp_le_u32 %[q], 2\ns_cbranch_scc1 2f\n"                            \
    "s_add_u32 %[wo], %[wo], 64\n" RE_LOAD_LONG(next)                                          \
    "2:\n.set re_w, " #r "\n.set re_u, " #r "+16\n" RE_HALF(C, P, X, Y, c)
#define RE_SGPRS                                                                                            \
    "s36", "s37", "s38", "s39", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49", "s50", \
        "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s64",   \
        "s65", "s66", "s67", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78",   \
        "s79", "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s92",   \
        "s93", "s94", "s95", "s96", "s97", "s98", "s99"
#define RE_ACC1 [acc0] "+v"(acc[0])
#define RE_ACC2 [acc0] "+v"(acc[0]), [acc1] "+v"(acc[1])
// NR rows for each of P points from base on; L: SHORT or LONG
#define RE_ASM(NR, P, base, X, Y, C, L, ...)                                                                \
    asm volatile("s_mov_b32 %[m], m0\n"                                                                     \
                 "global_load_dwordx2 %[c0], %[vo], %[cp]\n" RE_COEFS("%[c1]") RE_LOAD_##L(36)               \
                 ".set re_i, 0\n.rept " #NR "*" #P "\n"                                                      \
                 "ds_read_b64 v[" #base "+2*re_i:" #base "+1+2*re_i], %[xa] offset:512*re_i\n"               \
                 ".set re_i, re_i+1\n.endr\n.set re_u, 0\n"                                                  \
                 "1:\n" RE_SET_##L(C, P, X, Y, 36, 68, "%[c0]") RE_SET_##L(C, P, X, Y, 68, 36, "%[c1]")       \
                 "s_branch 1b\n9:\ns_waitcnt vmcnt(0) lgkmcnt(0)\ns_mov_b32 m0, %[m]\n"                       \
                 : RE_ACC##P, [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [c0] "=&v"(c0), [c1] "=&v"(c1), [vo] "+v"(vo),            \
                   [q] "+s"(q), [wo] "+s"(wo), [wo2] "+s"(wo2), [m] "=&s"(m0)                                \
                 : [wp] "s"(wp), [up] "s"(up), [cp] "s"(cp), [xa] "v"(xa), [vm] "v"(vm)                      \
                 : "memory", "scc", RE_SGPRS, __VA_ARGS__)
#define RE_VGPRS24 \
    "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", \
    "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", "v72", "v73", \
    "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85", "v86", "v87", \
    "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", "v100", "v101", \
    "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", \
    "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127"
#define RE_VGPRS56 \
    "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", \
    "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", "v72", "v73", \
    "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85", "v86", "v87", \
    "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", "v100", "v101", \
    "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", \
    "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", \
    "v130", "v131", "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", \
    "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", "v156", "v157", \
    "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", \
    "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", \
    "v186", "v187", "v188", "v189", "v190", "v191", "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", \
    "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", "v208", "v209", "v210", "v211", "v212", "v213", \
    "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", "v224", "v225", "v226", "v227", \
    "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237", "v238", "v239", "v240", "v241", \
    "v242", "v243", "v244", "v245", "v246", "v247", "v248", "v249", "v250", "v251", "v252", "v253", "v254", "v255"
#define RE_VGPRS113 \
    "v30", "v31", "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", \
    "v44", "v45", "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", \
    "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85", \
    "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", \
    "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113", \
    "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", \
    "v128", "v129", "v130", "v131", "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", \
    "v142", "v143", "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", \
    "v156", "v157", "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", \
    "v170", "v171", "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", \
    "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", "v192", "v193", "v194", "v195", "v196", "v197", \
    "v198", "v199", "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", "v208", "v209", "v210", "v211", \
    "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", "v224", "v225", \
    "v226", "v227", "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237", "v238", "v239", \
    "v240", "v241", "v242", "v243", "v244", "v245", "v246", "v247", "v248", "v249", "v250", "v251", "v252", "v253", \
    "v254", "v255"

constexpr int RE_MAX_N = 112;
constexpr int RE_WORD_PAD = 32;   // words that may be read (and not used) past a plane's end

// The register sets by number of variables: rows of the coordinate tile (n +
// 1 of them are used), and points that a lane holds.  Two points up to 55
// variables, whatever the number of points: with half of the lanes' second
// points unused a term still costs less than from LDS.
__host__ __device__ constexpr int regeval_rows(int n) { return n < 24 ? 24 : (n < 56 ? 56 : 113); }
__host__ __device__ constexpr int regeval_points(int rows) { return rows > 56 ? 1 : 2; }

// Whether `terms` terms of degree class md in `ranges` ranges (a polynomial's
// terms or a segment of them) are evaluated from registers.  A range costs the
// load of all rows, the wait for the first terms and a few terms from LDS at
// its end, with two waves on a SIMD to hide them (four up to 23 variables), so
// short ranges stay in LDS.  Measured at 1,024 points, registers / LDS, at
// ranges just above and below the line: 20 variables, degree 3: 38 terms 208 /
// 233 us, 19 terms 278 / 250 us; 40 variables, degree 4: 85 terms 90 / 93 us,
// 32 terms 121 / 99 us; 100 variables, degree 4: 781 terms (8,192 points) 227 /
// 364 us, 93 terms 122 / 107 us.  Past degree class 4 the LDS form takes a
// term's record apart lane by lane and the line lies lower, from 2^28 terms
// times points on; but it reads only the factor words that a term's own degree
// needs, and the registers all of the class's, so the line is that of terms of
// every degree up to the class's.  2,048 points, 2^28 terms times points,
// registers / LDS, for degrees 0 to 6, then for 6 alone: 20 variables, 16 terms
// 217 / 266, 221 / 321 us, 12 terms 295 / 250, 298 / 321; 40 variables, 48
// terms 230 / 242, 234 / 301, 32 terms 251 / 236, 257 / 299; 60 variables, 100
// terms 236 / 236, 240 / 304, 64 terms 246 / 239, 247 / 295.  None does below
// 2^26: the host knows neither the degree nor the number of derivative terms,
// and the launch of a kernel that turns out not to run would be more than 2% of
// the call.
__host__ __device__ inline bool regeval_pays(int n, uint32_t md, int64_t terms, int64_t ranges, int64_t N)
{
    if (n > RE_MAX_N || md > 8 || terms * N < ((int64_t)1 << 26)) return false;
    const int rows = regeval_rows(n);
    const bool low = md > 4 && terms * N >= ((int64_t)1 << 28);
    const int range = low ? (rows == 24 ? 16 : (rows == 56 ? 40 : 96)) : (rows == 24 ? 40 : (rows == 56 ? 80 : 384));
    return terms >= ranges * range;
}

// a 64-bit value that is the same on every lane, as a scalar
__device__ inline int64_t uniform_i64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// acc[p] += the sum of 8 q terms (1 <= q < 2^24) at point p of the lane:
// factor words from wp (and, for more than four factors, up), coefficients
// from cp, each term the product of C factors.  xa: LDS byte address of this
// lane's column of the coordinate tile (512 bytes per row, the points' tiles
// one after the other).  Every lane of the wave takes part.
template <int NR, int C>
__device__ inline void term_octets(double (&acc)[regeval_points(NR)], uint32_t q, const uint32_t *wp,
                                   const uint32_t *up, const double *cp, uint32_t xa)
{
    wp = reinterpret_cast<const uint32_t *>(uniform_i64(reinterpret_cast<int64_t>(wp)));
    up = reinterpret_cast<const uint32_t *>(uniform_i64(reinterpret_cast<int64_t>(up)));
    cp = reinterpret_cast<const double *>(uniform_i64(reinterpret_cast<int64_t>(cp)));
    q = (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
    double t0, t1, t2, t3, c0, c1;
    const uint32_t vm = 64u * q - 8u;
    uint32_t vo = 8u * (lane_id() & 15);
    vo = vo < vm ? vo : vm;
    uint32_t wo = 0, wo2 = 64, m0;
    if constexpr (NR == 24) {
        if constexpr (C == 2) RE_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 2, SHORT, RE_VGPRS24);
        if constexpr (C == 3) RE_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 3, SHORT, RE_VGPRS24);
        if constexpr (C == 4) RE_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 4, SHORT, RE_VGPRS24);
        if constexpr (C == 5) RE_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 5, LONG, RE_VGPRS24);
        if constexpr (C == 6) RE_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 6, LONG, RE_VGPRS24);
        if constexpr (C == 8) RE_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 8, LONG, RE_VGPRS24);
    }
    if constexpr (NR == 56) {
        if constexpr (C == 2) RE_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 2, SHORT, RE_VGPRS56);
        if constexpr (C == 3) RE_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 3, SHORT, RE_VGPRS56);
        if constexpr (C == 4) RE_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 4, SHORT, RE_VGPRS56);
        if constexpr (C == 5) RE_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 5, LONG, RE_VGPRS56);
        if constexpr (C == 6) RE_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 6, LONG, RE_VGPRS56);
        if constexpr (C == 8) RE_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 8, LONG, RE_VGPRS56);
    }
    if constexpr (NR == 113) {
        if constexpr (C == 2) RE_ASM(113, 1, 30, "v[30:31]", "", 2, SHORT, RE_VGPRS113);
        if constexpr (C == 3) RE_ASM(113, 1, 30, "v[30:31]", "", 3, SHORT, RE_VGPRS113);
        if constexpr (C == 4) RE_ASM(113, 1, 30, "v[30:31]", "", 4, SHORT, RE_VGPRS113);
        if constexpr (C == 5) RE_ASM(113, 1, 30, "v[30:31]", "", 5, LONG, RE_VGPRS113);
        if constexpr (C == 6) RE_ASM(113, 1, 30, "v[30:31]", "", 6, LONG, RE_VGPRS113);
        if constexpr (C == 8) RE_ASM(113, 1, 30, "v[30:31]", "", 8, LONG, RE_VGPRS113);
    }
}

// ---- one sum over points per term (dC), 64 terms at a time
//
// The products of four terms are weighted by the lane's point and added over
// the wave down to 16 partial sums each, the four terms' in one register: two
// exchanges of half waves (v_permlane32_swap) and one of rows of 16
// (v_permlane16_swap), three additions.  The partial sums go to the wave's LDS
// buffer, 17 doubles per term so that the reads meet no bank twice; after 64
// terms each lane adds those of its own.  v[22:29] hold the products, v[30:31]
// the first half of four terms at two points per lane.
#define RD_SWAP(w, a, b) "v_permlane" w "_swap_b32 v" #a ", v" #b "\n"
#define RD_OUT "ds_write_b64 %[wa], v[22:23] offset:544*re_q\n.set re_q, re_q+1\n"
// v[22:23] = its own and v[24:25]'s sums over half waves
#define RD_HALF "s_nop 1\n" RD_SWAP("32", 22, 24) RD_SWAP("32", 23, 25) "v_add_f64 v[22:23], v[22:23], v[24:25]\n"
#define RD_LAST1                                                                                       \
    "s_set_gpr_idx_off\nv_mul_f64 %[t0], %[t0], %[g0]\nv_mul_f64 %[t1], %[t1], %[g0]\n"                  \
    "v_mul_f64 %[t2], %[t2], %[g0]\nv_mul_f64 %[t3], %[t3], %[g0]\n" RD_HALF                            \
    RD_SWAP("32", 26, 28) RD_SWAP("32", 27, 29) "v_add_f64 v[26:27], v[26:27], v[28:29]\ns_nop 1\n"      \
    RD_SWAP("16", 22, 26) RD_SWAP("16", 23, 27) "v_add_f64 v[22:23], v[22:23], v[26:27]\n" RD_OUT        \
    ".set re_w, re_w+4\n.set re_u, re_u+4\n"
#define RD_WEIGH2                                                                                      \
    "s_set_gpr_idx_off\nv_mul_f64 %[t0], %[t0], %[g0]\nv_mul_f64 %[t2], %[t2], %[g0]\n"                  \
    "v_fma_f64 v[22:23], v[24:25], %[g1], v[22:23]\nv_fma_f64 v[24:25], v[28:29], %[g1], v[26:27]\n" RD_HALF \
    ".set re_w, re_w+2\n.set re_u, re_u+2\n"
#define RD_FOUR1(C, X, Y) RE_LIST##C(1, X, Y) RD_LAST1
#define RD_FOUR2(C, X, Y)                                                                              \
    RE_LIST##C(2, X, Y) RD_WEIGH2 "v_mov_b32 v30, v22\nv_mov_b32 v31, v23\n" RE_LIST##C(2, X, Y) RD_WEIGH2 \
    "s_nop 1\n" RD_SWAP("16", 30, 22) RD_SWAP("16", 31, 23) "v_add_f64 v[22:23], v[30:31], v[22:23]\n" RD_OUT
#define RD_OCTET(C, P, X, Y) \
    "s_sub_u32 %[q], %[q], 1\ns_cbranch_scc1 9f\n.rept 2\n" RD_FOUR##P(C, X, Y) ".endr\n"
#define RD_SET_SHORT(C, P, X, Y, r, next)                                                              \
    "s_waitcnt lgkmcnt(0)\ns_cmp_le_u32 %[q], 4\ns_cbranch_scc1 2f\n"                                    \
    "s_add_u32 %[wo], %[wo], 128\ns_add_u32 %[wo2], %[wo2], 128\n" RE_LOAD_SHORT(next)                  \
    "2:\n.set re_w, " #r "\n" RD_OCTET(C, P, X, Y) RD_OCTET(C, P, X, Y) RD_OCTET(C, P, X, Y) RD_OCTET(C, P, X, Y)
#define RD_SET_LONG(C, P, X, Y, r, next)                                                               \
    "s_waitcnt lgkmcnt(0)\ns_cmp_le_u32 %[q], 2\ns_cbranch_scc1 2f\n"                                    \
    "s_add_u32 %[wo], %[wo], 64\n" RE_LOAD_LONG(next)                                                  \
    "2:\n.set re_w, " #r "\n.set re_u, " #r "+16\n" RD_OCTET(C, P, X, Y) RD_OCTET(C, P, X, Y)
#define RD_BATCH_SHORT(C, P, X, Y) RD_SET_SHORT(C, P, X, Y, 36, 68) RD_SET_SHORT(C, P, X, Y, 68, 36)
#define RD_BATCH_LONG(C, P, X, Y)                                                                      \
    RD_SET_LONG(C, P, X, Y, 36, 68) RD_SET_LONG(C, P, X, Y, 68, 36) RD_SET_LONG(C, P, X, Y, 36, 68)      \
        RD_SET_LONG(C, P, X, Y, 68, 36)
// the lane's 16 partial sums, in order, and the store of those within the range
#define RD_READ(o)                                                                                     \
    "ds_read_b64 v[22:23], %[ra] offset:" #o "\nds_read_b64 v[24:25], %[ra] offset:" #o "+8\n"           \
    "ds_read_b64 v[26:27], %[ra] offset:" #o "+16\nds_read_b64 v[28:29], %[ra] offset:" #o "+24\n"       \
    "s_waitcnt lgkmcnt(0)\n"
#define RD_SUM \
    "v_add_f64 %[acc], %[acc], v[22:23]\nv_add_f64 %[acc], %[acc], v[24:25]\nv_add_f64 %[acc], %[acc], v[26:27]\n" \
    "v_add_f64 %[acc], %[acc], v[28:29]\n"
#define RD_FLUSH                                                                                       \
    "s_waitcnt lgkmcnt(0)\n" RD_READ(0)                             \
    "v_add_f64 %[acc], v[22:23], v[24:25]\nv_add_f64 %[acc], %[acc], v[26:27]\n"                         \
    "v_add_f64 %[acc], %[acc], v[28:29]\n" RD_READ(32) RD_SUM RD_READ(64) RD_SUM RD_READ(96) RD_SUM      \
    "v_cmp_gt_u32 vcc, %[vend], %[vo]\ns_and_saveexec_b64 %[ex], vcc\n"                                  \
    "global_store_dwordx2 %[vo], %[acc], %[op]\ns_mov_b64 exec, %[ex]\nv_add_u32 %[vo], 0x200, %[vo]\n"
#define RD_G1 [g0] "v"(g[0])
#define RD_G2 [g0] "v"(g[0]), [g1] "v"(g[1])
#define RD_ASM(NR, P, base, X, Y, C, L, ...)                                                                \
    asm volatile("s_mov_b32 %[m], m0\n" RE_LOAD_##L(36)                                                     \
                 ".set re_i, 0\n.rept " #NR "*" #P "\n"                                                      \
                 "ds_read_b64 v[" #base "+2*re_i:" #base "+1+2*re_i], %[xa] offset:512*re_i\n"               \
                 ".set re_i, re_i+1\n.endr\n.set re_u, 0\n"                                                  \
                 "1:\n.set re_q, 0\n" RD_BATCH_##L(C, P, X, Y) RD_FLUSH "s_branch 1b\n"                       \
                 "9:\n" RD_FLUSH "s_waitcnt vmcnt(0) lgkmcnt(0)\ns_mov_b32 m0, %[m]\n"                        \
                 : [t0] "=&{v[22:23]}"(t0), [t1] "=&{v[24:25]}"(t1), [t2] "=&{v[26:27]}"(t2),                \
                   [t3] "=&{v[28:29]}"(t3), [acc] "=&v"(acc), [vo] "+v"(vo), [q] "+s"(q), [wo] "+s"(wo),     \
                   [wo2] "+s"(wo2), [m] "=&s"(m0), [ex] "=&s"(ex)                                            \
                 : [wp] "s"(wp), [up] "s"(up), [op] "s"(op), [xa] "v"(xa), [wa] "v"(wa), [ra] "v"(ra),       \
                   [vend] "v"(vend), RD_G##P                                                                 \
                 : "memory", "scc", "vcc", RE_SGPRS, __VA_ARGS__)

// Doubles of a wave's buffer: 64 terms of 16 partial sums and a spare.
constexpr int RD_BUF = 64 * 17;

// out[t] = the sum over the wave's points p of g[p] * term t at p, for 8 q
// terms (1 <= q < 2^23), coefficients left out.  buf: LDS byte address of the
// wave's buffer.  The rest as in term_octets.
template <int NR, int C>
__device__ inline void dc_octets(double *out, uint32_t q, const uint32_t *wp, const uint32_t *up, uint32_t xa,
                                 const double (&g)[regeval_points(NR)], uint32_t buf)
{
    wp = reinterpret_cast<const uint32_t *>(uniform_i64(reinterpret_cast<int64_t>(wp)));
    up = reinterpret_cast<const uint32_t *>(uniform_i64(reinterpret_cast<int64_t>(up)));
    double *op = reinterpret_cast<double *>(uniform_i64(reinterpret_cast<int64_t>(out)));
    q = (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
    double t0, t1, t2, t3, acc;
    const uint32_t lane = (uint32_t)lane_id(), vend = 64u * q;
    const uint32_t wa = buf + (lane >> 4) * 136u + (lane & 15u) * 8u, ra = buf + lane * 136u;
    // the exchanges leave terms 0, 2, 1, 3 in the rows of 16
    uint32_t vo = 8u * ((lane & ~3u) + ((lane & 1u) << 1) + ((lane >> 1) & 1u));
    uint32_t wo = 0, wo2 = 64, m0;
    uint64_t ex;
    if constexpr (NR == 24) {
        if constexpr (C == 2) RD_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 2, SHORT, "v30", "v31", RE_VGPRS24);
        if constexpr (C == 3) RD_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 3, SHORT, "v30", "v31", RE_VGPRS24);
        if constexpr (C == 4) RD_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 4, SHORT, "v30", "v31", RE_VGPRS24);
        if constexpr (C == 5) RD_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 5, LONG, "v30", "v31", RE_VGPRS24);
        if constexpr (C == 6) RD_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 6, LONG, "v30", "v31", RE_VGPRS24);
        if constexpr (C == 8) RD_ASM(24, 2, 32, "v[32:33]", "v[80:81]", 8, LONG, "v30", "v31", RE_VGPRS24);
    }
    if constexpr (NR == 56) {
        if constexpr (C == 2) RD_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 2, SHORT, "v30", "v31", RE_VGPRS56);
        if constexpr (C == 3) RD_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 3, SHORT, "v30", "v31", RE_VGPRS56);
        if constexpr (C == 4) RD_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 4, SHORT, "v30", "v31", RE_VGPRS56);
        if constexpr (C == 5) RD_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 5, LONG, "v30", "v31", RE_VGPRS56);
        if constexpr (C == 6) RD_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 6, LONG, "v30", "v31", RE_VGPRS56);
        if constexpr (C == 8) RD_ASM(56, 2, 32, "v[32:33]", "v[144:145]", 8, LONG, "v30", "v31", RE_VGPRS56);
    }
    if constexpr (NR == 113) {
        if constexpr (C == 2) RD_ASM(113, 1, 30, "v[30:31]", "", 2, SHORT, RE_VGPRS113);
        if constexpr (C == 3) RD_ASM(113, 1, 30, "v[30:31]", "", 3, SHORT, RE_VGPRS113);
        if constexpr (C == 4) RD_ASM(113, 1, 30, "v[30:31]", "", 4, SHORT, RE_VGPRS113);
        if constexpr (C == 5) RD_ASM(113, 1, 30, "v[30:31]", "", 5, LONG, RE_VGPRS113);
        if constexpr (C == 6) RD_ASM(113, 1, 30, "v[30:31]", "", 6, LONG, RE_VGPRS113);
        if constexpr (C == 8) RD_ASM(113, 1, 30, "v[30:31]", "", 8, LONG, RE_VGPRS113);
    }
}

}  // namespace polyhip
