// Register-tiled backward kernel (see sspmm_bwd_regs.hip), one translation unit per storage format of dY.
//
// Bound by instruction issue.  A SIMD retires a vector instruction in 5.2 clocks and a scalar one in 4.7, side by side from its two
// wavefronts, a wavefront alone one of either in 4.6 to 5; a step of 115 M entries on 233 k nodes, k = 32, has 18 pairs of entries a wavefront:
// 3.2 ms with the records read by v_readlane at a counted lane (9.3 clocks each), 2.4 with DPP broadcasts and constant lanes.  The row copies
// alone take 1.4 ms there, 2.2 at k = 64 (1.15 with bf16 dY).
#pragma once

#include "common.hpp"

namespace maxk {
namespace {

struct RegsArgs {
    const void* dY;
    const void* sp_index;
    float* dXs;
    const uint4* rec;        // {accumulator | LDS address of the row; weight} twice: two entries of a wavefront's list
    const uint32_t* hdr;     // [steps * 8 wavefronts][HD] {first record, batches, rows to load}
    const int32_t* node;     // [sets * 8 wavefronts * slots * groups] destination of an accumulator, or -1
    const int32_t* row;      // ... the row that its sum goes to: of dXs, from N on of `extra`
    float* extra;
    int64_t N;
    const RegsUnit* unit;    // one per workgroup
    const RegsPart* part;
    float* parts;            // sums that left: of a part [8 wavefronts][its accumulators][64 lanes]
    uint32_t row_bytes;
    int32_t k, index_bytes;
};

typedef float regs_v32 __attribute__((ext_vector_type(32)));
typedef float regs_v16 __attribute__((ext_vector_type(16)));

// The accumulators (v32..v143) and the LDS offsets of their columns (v144..v255) stay in these registers for the whole
// kernel: the instructions that use them add the number of the accumulator to the register number (VGPR index mode), which
// needs consecutive registers with a known first one.
#define MAXK_REGS_FILE                                                                                                \
    "+{v[32:63]}"(A0), "+{v[64:95]}"(A1), "+{v[96:127]}"(A2), "+{v[128:143]}"(A3), "+{v[144:159]}"(C0), "+{v[160:191]}"(C1), \
        "+{v[192:223]}"(C2), "+{v[224:255]}"(C3)

// A list is worked on in batches of slots; a slot has an entry for each lane group.  Its records sit in registers, 16 slots (a
// chunk) in a pair of them: lane l holds the record of slot l % 16 of its own group, {LDS address of the row | accumulator;
// weight}, and an instruction takes slot e from it by a DPP broadcast within rows of 16 lanes.  Only the accumulators' numbers
// have to be scalar.
#define RL(S, M, L) "v_readlane_b32 " S ", " M ", " L "\n"
#define SLOT(E) " row_newbcast:" E " row_mask:0xf bank_mask:0xf\n"
#define AT(D, M, E) "v_add_u32_dpp " D ", " M ", v144" SLOT(E)
#define AT2(D, M, E) "v_add_u32_dpp " D ", " M ", v145" SLOT(E)
#define MAD(D, X, E) "v_fmac_f32_dpp v32, " X ", " D SLOT(E)
#define MAD2(D, X, E) "v_fmac_f32_dpp v33, " X ", " D SLOT(E)
#define ON_C(S) "s_set_gpr_idx_on " S ", 2\n"  // adds S to the register number of the second source
#define ON_A(S) "s_set_gpr_idx_on " S ", 12\n" // ... of the third source and of the destination
#define IDX(S) "s_set_gpr_idx_idx " S "\n"
#define OFF "s_set_gpr_idx_off\n"
#define LANES(N, FROM) "s_bfm_b64 exec, " N ", " FROM "\n"
#define ALL "s_mov_b64 exec, -1\n"

// One batch in two halves.  ADDR: the accumulators' numbers, LDS addresses, the LDS reads under way.  FMA: what they brought,
// times the weights, into the accumulators.  (All lanes add up a first address, the later lane groups then their own.)  S0..S7: scalar registers of the batch, D0..D3: its data, M and X: the records,
// E0..E3: slots.
// one destination a register (32 < k <= 64): four entries
#define ADDR_1(LD, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1, E2, E3)                                        \
    RL(S0, M, E0) RL(S1, M, E1) RL(S2, M, E2) RL(S3, M, E3)                                                                   \
    ON_C(S0) AT(D0, M, E0) LD(D0) IDX(S1) AT(D1, M, E1) LD(D1) IDX(S2) AT(D2, M, E2) LD(D2) IDX(S3) AT(D3, M, E3) LD(D3) LD##_END
#define FMA_1(CV, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1, E2, E3)                                         \
    CV(D0) CV(D1) CV(D2) CV(D3)                                                                                               \
    ON_A(S0) MAD(D0, X, E0) IDX(S1) MAD(D1, X, E1) IDX(S2) MAD(D2, X, E2) IDX(S3) MAD(D3, X, E3) OFF
// two registers a destination (k > 64): two entries
#define ADDR_W(LD, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1)                                                \
    RL(S0, M, E0) RL(S1, M, E1)                                                                                               \
    ON_C(S0) AT(D0, M, E0) LD(D0) AT2(D1, M, E0) LD(D1) IDX(S1) AT(D2, M, E1) LD(D2) AT2(D3, M, E1) LD(D3) LD##_END
#define FMA_W(CV, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1)                                                 \
    CV(D0) CV(D1) CV(D2) CV(D3)                                                                                               \
    ON_A(S0) MAD(D0, X, E0) MAD2(D1, X, E0) IDX(S1) MAD(D2, X, E1) MAD2(D3, X, E1) OFF
// two destinations a register (16 < k <= 32): four pairs
#define ADDR_2(LD, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1, E2, E3)                                        \
    RL(S0, M, E0) RL(S1, M, E1) RL(S2, M, E2) RL(S3, M, E3) RL(S4, M, "32+" E0) RL(S5, M, "32+" E1) RL(S6, M, "32+" E2) RL(S7, M, "32+" E3) \
    ON_C(S0) AT(D0, M, E0) IDX(S1) AT(D1, M, E1) IDX(S2) AT(D2, M, E2) IDX(S3) AT(D3, M, E3)                   \
    LANES("32", "32") IDX(S4) AT(D0, M, E0) IDX(S5) AT(D1, M, E1) IDX(S6) AT(D2, M, E2) IDX(S7) AT(D3, M, E3) LD##_END          \
    ALL LD(D0) LD(D1) LD(D2) LD(D3)
#define FMA_2(CV, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1, E2, E3)                                         \
    CV(D0) CV(D1) CV(D2) CV(D3)                                                                                               \
    LANES("32", "0") ON_A(S0) MAD(D0, X, E0) IDX(S1) MAD(D1, X, E1) IDX(S2) MAD(D2, X, E2) IDX(S3) MAD(D3, X, E3)               \
    LANES("32", "32") IDX(S4) MAD(D0, X, E0) IDX(S5) MAD(D1, X, E1) IDX(S6) MAD(D2, X, E2) IDX(S7) MAD(D3, X, E3) OFF ALL
// four destinations a register (k <= 16): two quads
#define ADDR_4(LD, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1)                                                \
    RL(S0, M, E0) RL(S1, M, E1) RL(S2, M, "16+" E0) RL(S3, M, "16+" E1) RL(S4, M, "32+" E0) RL(S5, M, "32+" E1) RL(S6, M, "48+" E0) RL(S7, M, "48+" E1) \
    ON_C(S0) AT(D0, M, E0) IDX(S1) AT(D1, M, E1) LANES("16", "16") IDX(S2) AT(D0, M, E0) IDX(S3) AT(D1, M, E1)  \
    LANES("16", "32") IDX(S4) AT(D0, M, E0) IDX(S5) AT(D1, M, E1) LANES("16", "48") IDX(S6) AT(D0, M, E0) IDX(S7) AT(D1, M, E1) LD##_END \
    ALL LD(D0) LD(D1)
#define FMA_4(CV, S0, S1, S2, S3, S4, S5, S6, S7, D0, D1, D2, D3, M, X, E0, E1)                                                 \
    CV(D0) CV(D1)                                                                                                             \
    LANES("16", "0") ON_A(S0) MAD(D0, X, E0) IDX(S1) MAD(D1, X, E1) LANES("16", "16") IDX(S2) MAD(D0, X, E0) IDX(S3) MAD(D1, X, E1) \
    LANES("16", "32") IDX(S4) MAD(D0, X, E0) IDX(S5) MAD(D1, X, E1) LANES("16", "48") IDX(S6) MAD(D0, X, E0) IDX(S7) MAD(D1, X, E1) OFF ALL

#define LD_F32(D) "ds_read_b32 " D ", " D "\n"
#define LD_16(D) "ds_read_u16 " D ", " D "\n"
#define LD_F32_END ""  // the next vector instruction sets its own mode
#define LD_16_END OFF  // ... is a conversion
#define CV_F32(D) ""
#define CV_BF16(D) "v_lshlrev_b32 " D ", 16, " D "\n"
#define CV_F16(D) "v_cvt_f32_f16 " D ", " D "\n"

// Two sets of registers take turns, so that the LDS reads of a batch are under way while the one before is added.  Straight
// code, left after the last batch of the list: batch b + 1 is begun (registers of set B, slots F) before batch b is added.
#define SET_A "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "v24", "v25", "v26", "v27"
#define SET_B "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "v28", "v29", "v30", "v31"
#define CALL(F, ...) F(__VA_ARGS__)
#define MORE(ADDR, FMA, LD, CV, READS, B, S, Q, S2, Q2)                                                     \
    "s_sub_u32 s64, s64, 1\ns_cbranch_scc1 .Ltail" B "_%=\n" CALL(ADDR, LD, S2, Q2) "s_waitcnt lgkmcnt(" READS ")\n" CALL(FMA, CV, S, Q)
#define TAIL(FMA, CV, B, S, Q) ".Ltail" B "_%=:\ns_waitcnt lgkmcnt(0)\n" CALL(FMA, CV, S, Q) "s_branch .Lout_%=\n"
// slots of a batch: Q four, P two; first digit: chunk
#define Q00 "v16", "v17", "0", "1", "2", "3"
#define Q01 "v16", "v17", "4", "5", "6", "7"
#define Q02 "v16", "v17", "8", "9", "10", "11"
#define Q03 "v16", "v17", "12", "13", "14", "15"
#define Q10 "v18", "v19", "0", "1", "2", "3"
#define Q11 "v18", "v19", "4", "5", "6", "7"
#define Q12 "v18", "v19", "8", "9", "10", "11"
#define Q13 "v18", "v19", "12", "13", "14", "15"
#define Q20 "v20", "v21", "0", "1", "2", "3"
#define Q21 "v20", "v21", "4", "5", "6", "7"
#define Q22 "v20", "v21", "8", "9", "10", "11"
#define Q23 "v20", "v21", "12", "13", "14", "15"
#define Q30 "v22", "v23", "0", "1", "2", "3"
#define Q31 "v22", "v23", "4", "5", "6", "7"
#define Q32 "v22", "v23", "8", "9", "10", "11"
#define Q33 "v22", "v23", "12", "13", "14", "15"
#define P00 "v16", "v17", "0", "1"
#define P01 "v16", "v17", "2", "3"
#define P02 "v16", "v17", "4", "5"
#define P03 "v16", "v17", "6", "7"
#define P04 "v16", "v17", "8", "9"
#define P05 "v16", "v17", "10", "11"
#define P06 "v16", "v17", "12", "13"
#define P07 "v16", "v17", "14", "15"
#define P10 "v18", "v19", "0", "1"
#define P11 "v18", "v19", "2", "3"
#define P12 "v18", "v19", "4", "5"
#define P13 "v18", "v19", "6", "7"
#define P14 "v18", "v19", "8", "9"
#define P15 "v18", "v19", "10", "11"
#define P16 "v18", "v19", "12", "13"
#define P17 "v18", "v19", "14", "15"
#define P20 "v20", "v21", "0", "1"
#define P21 "v20", "v21", "2", "3"
#define P22 "v20", "v21", "4", "5"
#define P23 "v20", "v21", "6", "7"
#define P24 "v20", "v21", "8", "9"
#define P25 "v20", "v21", "10", "11"
#define P26 "v20", "v21", "12", "13"
#define P27 "v20", "v21", "14", "15"
#define P30 "v22", "v23", "0", "1"
#define P31 "v22", "v23", "2", "3"
#define P32 "v22", "v23", "4", "5"
#define P33 "v22", "v23", "6", "7"
#define P34 "v22", "v23", "8", "9"
#define P35 "v22", "v23", "10", "11"
#define P36 "v22", "v23", "12", "13"
#define P37 "v22", "v23", "14", "15"
#define BATCHES_Q2(ADDR, FMA, LD, CV, READS) \
    CALL(ADDR, LD, SET_A, Q00) \
    MORE(ADDR, FMA, LD, CV, READS, "0", SET_A, Q00, SET_B, Q01) \
    MORE(ADDR, FMA, LD, CV, READS, "1", SET_B, Q01, SET_A, Q02) \
    MORE(ADDR, FMA, LD, CV, READS, "2", SET_A, Q02, SET_B, Q03) \
    MORE(ADDR, FMA, LD, CV, READS, "3", SET_B, Q03, SET_A, Q10) \
    MORE(ADDR, FMA, LD, CV, READS, "4", SET_A, Q10, SET_B, Q11) \
    MORE(ADDR, FMA, LD, CV, READS, "5", SET_B, Q11, SET_A, Q12) \
    MORE(ADDR, FMA, LD, CV, READS, "6", SET_A, Q12, SET_B, Q13) \
    TAIL(FMA, CV, "7", SET_B, Q13) \
    TAIL(FMA, CV, "6", SET_A, Q12) \
    TAIL(FMA, CV, "5", SET_B, Q11) \
    TAIL(FMA, CV, "4", SET_A, Q10) \
    TAIL(FMA, CV, "3", SET_B, Q03) \
    TAIL(FMA, CV, "2", SET_A, Q02) \
    TAIL(FMA, CV, "1", SET_B, Q01) \
    TAIL(FMA, CV, "0", SET_A, Q00)
#define BATCHES_Q4(ADDR, FMA, LD, CV, READS) \
    CALL(ADDR, LD, SET_A, Q00) \
    MORE(ADDR, FMA, LD, CV, READS, "0", SET_A, Q00, SET_B, Q01) \
    MORE(ADDR, FMA, LD, CV, READS, "1", SET_B, Q01, SET_A, Q02) \
    MORE(ADDR, FMA, LD, CV, READS, "2", SET_A, Q02, SET_B, Q03) \
    MORE(ADDR, FMA, LD, CV, READS, "3", SET_B, Q03, SET_A, Q10) \
    MORE(ADDR, FMA, LD, CV, READS, "4", SET_A, Q10, SET_B, Q11) \
    MORE(ADDR, FMA, LD, CV, READS, "5", SET_B, Q11, SET_A, Q12) \
    MORE(ADDR, FMA, LD, CV, READS, "6", SET_A, Q12, SET_B, Q13) \
    MORE(ADDR, FMA, LD, CV, READS, "7", SET_B, Q13, SET_A, Q20) \
    MORE(ADDR, FMA, LD, CV, READS, "8", SET_A, Q20, SET_B, Q21) \
    MORE(ADDR, FMA, LD, CV, READS, "9", SET_B, Q21, SET_A, Q22) \
    MORE(ADDR, FMA, LD, CV, READS, "10", SET_A, Q22, SET_B, Q23) \
    MORE(ADDR, FMA, LD, CV, READS, "11", SET_B, Q23, SET_A, Q30) \
    MORE(ADDR, FMA, LD, CV, READS, "12", SET_A, Q30, SET_B, Q31) \
    MORE(ADDR, FMA, LD, CV, READS, "13", SET_B, Q31, SET_A, Q32) \
    MORE(ADDR, FMA, LD, CV, READS, "14", SET_A, Q32, SET_B, Q33) \
    TAIL(FMA, CV, "15", SET_B, Q33) \
    TAIL(FMA, CV, "14", SET_A, Q32) \
    TAIL(FMA, CV, "13", SET_B, Q31) \
    TAIL(FMA, CV, "12", SET_A, Q30) \
    TAIL(FMA, CV, "11", SET_B, Q23) \
    TAIL(FMA, CV, "10", SET_A, Q22) \
    TAIL(FMA, CV, "9", SET_B, Q21) \
    TAIL(FMA, CV, "8", SET_A, Q20) \
    TAIL(FMA, CV, "7", SET_B, Q13) \
    TAIL(FMA, CV, "6", SET_A, Q12) \
    TAIL(FMA, CV, "5", SET_B, Q11) \
    TAIL(FMA, CV, "4", SET_A, Q10) \
    TAIL(FMA, CV, "3", SET_B, Q03) \
    TAIL(FMA, CV, "2", SET_A, Q02) \
    TAIL(FMA, CV, "1", SET_B, Q01) \
    TAIL(FMA, CV, "0", SET_A, Q00)
#define BATCHES_P1(ADDR, FMA, LD, CV, READS) \
    CALL(ADDR, LD, SET_A, P00) \
    MORE(ADDR, FMA, LD, CV, READS, "0", SET_A, P00, SET_B, P01) \
    MORE(ADDR, FMA, LD, CV, READS, "1", SET_B, P01, SET_A, P02) \
    MORE(ADDR, FMA, LD, CV, READS, "2", SET_A, P02, SET_B, P03) \
    MORE(ADDR, FMA, LD, CV, READS, "3", SET_B, P03, SET_A, P04) \
    MORE(ADDR, FMA, LD, CV, READS, "4", SET_A, P04, SET_B, P05) \
    MORE(ADDR, FMA, LD, CV, READS, "5", SET_B, P05, SET_A, P06) \
    MORE(ADDR, FMA, LD, CV, READS, "6", SET_A, P06, SET_B, P07) \
    TAIL(FMA, CV, "7", SET_B, P07) \
    TAIL(FMA, CV, "6", SET_A, P06) \
    TAIL(FMA, CV, "5", SET_B, P05) \
    TAIL(FMA, CV, "4", SET_A, P04) \
    TAIL(FMA, CV, "3", SET_B, P03) \
    TAIL(FMA, CV, "2", SET_A, P02) \
    TAIL(FMA, CV, "1", SET_B, P01) \
    TAIL(FMA, CV, "0", SET_A, P00)
#define BATCHES_P4(ADDR, FMA, LD, CV, READS) \
    CALL(ADDR, LD, SET_A, P00) \
    MORE(ADDR, FMA, LD, CV, READS, "0", SET_A, P00, SET_B, P01) \
    MORE(ADDR, FMA, LD, CV, READS, "1", SET_B, P01, SET_A, P02) \
    MORE(ADDR, FMA, LD, CV, READS, "2", SET_A, P02, SET_B, P03) \
    MORE(ADDR, FMA, LD, CV, READS, "3", SET_B, P03, SET_A, P04) \
    MORE(ADDR, FMA, LD, CV, READS, "4", SET_A, P04, SET_B, P05) \
    MORE(ADDR, FMA, LD, CV, READS, "5", SET_B, P05, SET_A, P06) \
    MORE(ADDR, FMA, LD, CV, READS, "6", SET_A, P06, SET_B, P07) \
    MORE(ADDR, FMA, LD, CV, READS, "7", SET_B, P07, SET_A, P10) \
    MORE(ADDR, FMA, LD, CV, READS, "8", SET_A, P10, SET_B, P11) \
    MORE(ADDR, FMA, LD, CV, READS, "9", SET_B, P11, SET_A, P12) \
    MORE(ADDR, FMA, LD, CV, READS, "10", SET_A, P12, SET_B, P13) \
    MORE(ADDR, FMA, LD, CV, READS, "11", SET_B, P13, SET_A, P14) \
    MORE(ADDR, FMA, LD, CV, READS, "12", SET_A, P14, SET_B, P15) \
    MORE(ADDR, FMA, LD, CV, READS, "13", SET_B, P15, SET_A, P16) \
    MORE(ADDR, FMA, LD, CV, READS, "14", SET_A, P16, SET_B, P17) \
    MORE(ADDR, FMA, LD, CV, READS, "15", SET_B, P17, SET_A, P20) \
    MORE(ADDR, FMA, LD, CV, READS, "16", SET_A, P20, SET_B, P21) \
    MORE(ADDR, FMA, LD, CV, READS, "17", SET_B, P21, SET_A, P22) \
    MORE(ADDR, FMA, LD, CV, READS, "18", SET_A, P22, SET_B, P23) \
    MORE(ADDR, FMA, LD, CV, READS, "19", SET_B, P23, SET_A, P24) \
    MORE(ADDR, FMA, LD, CV, READS, "20", SET_A, P24, SET_B, P25) \
    MORE(ADDR, FMA, LD, CV, READS, "21", SET_B, P25, SET_A, P26) \
    MORE(ADDR, FMA, LD, CV, READS, "22", SET_A, P26, SET_B, P27) \
    MORE(ADDR, FMA, LD, CV, READS, "23", SET_B, P27, SET_A, P30) \
    MORE(ADDR, FMA, LD, CV, READS, "24", SET_A, P30, SET_B, P31) \
    MORE(ADDR, FMA, LD, CV, READS, "25", SET_B, P31, SET_A, P32) \
    MORE(ADDR, FMA, LD, CV, READS, "26", SET_A, P32, SET_B, P33) \
    MORE(ADDR, FMA, LD, CV, READS, "27", SET_B, P33, SET_A, P34) \
    MORE(ADDR, FMA, LD, CV, READS, "28", SET_A, P34, SET_B, P35) \
    MORE(ADDR, FMA, LD, CV, READS, "29", SET_B, P35, SET_A, P36) \
    MORE(ADDR, FMA, LD, CV, READS, "30", SET_A, P36, SET_B, P37) \
    TAIL(FMA, CV, "31", SET_B, P37) \
    TAIL(FMA, CV, "30", SET_A, P36) \
    TAIL(FMA, CV, "29", SET_B, P35) \
    TAIL(FMA, CV, "28", SET_A, P34) \
    TAIL(FMA, CV, "27", SET_B, P33) \
    TAIL(FMA, CV, "26", SET_A, P32) \
    TAIL(FMA, CV, "25", SET_B, P31) \
    TAIL(FMA, CV, "24", SET_A, P30) \
    TAIL(FMA, CV, "23", SET_B, P27) \
    TAIL(FMA, CV, "22", SET_A, P26) \
    TAIL(FMA, CV, "21", SET_B, P25) \
    TAIL(FMA, CV, "20", SET_A, P24) \
    TAIL(FMA, CV, "19", SET_B, P23) \
    TAIL(FMA, CV, "18", SET_A, P22) \
    TAIL(FMA, CV, "17", SET_B, P21) \
    TAIL(FMA, CV, "16", SET_A, P20) \
    TAIL(FMA, CV, "15", SET_B, P17) \
    TAIL(FMA, CV, "14", SET_A, P16) \
    TAIL(FMA, CV, "13", SET_B, P15) \
    TAIL(FMA, CV, "12", SET_A, P14) \
    TAIL(FMA, CV, "11", SET_B, P13) \
    TAIL(FMA, CV, "10", SET_A, P12) \
    TAIL(FMA, CV, "9", SET_B, P11) \
    TAIL(FMA, CV, "8", SET_A, P10) \
    TAIL(FMA, CV, "7", SET_B, P07) \
    TAIL(FMA, CV, "6", SET_A, P06) \
    TAIL(FMA, CV, "5", SET_B, P05) \
    TAIL(FMA, CV, "4", SET_A, P04) \
    TAIL(FMA, CV, "3", SET_B, P03) \
    TAIL(FMA, CV, "2", SET_A, P02) \
    TAIL(FMA, CV, "1", SET_B, P01) \
    TAIL(FMA, CV, "0", SET_A, P00)
#define MAXK_REGS_LIST(BATCHES, ADDR, FMA, LD, CV, READS)                                                             \
    asm volatile("s_sub_u32 s64, %[n], 1\ns_cbranch_scc1 .Lout_%=\n" BATCHES(ADDR, FMA, LD, CV, READS) ".Lout_%=:\n"    \
                 : MAXK_REGS_FILE                                                                                     \
                 : [n] "s"(batches), "{v[16:17]}"(chunk[0]), "{v[18:19]}"(chunk[1]), "{v[20:21]}"(chunk[2]), "{v[22:23]}"(chunk[3])  \
                 : "memory", "scc", "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "s48", "s49", "s50", "s51", "s52", "s53", \
                   "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s64")

// 16 bytes a lane from `from` to LDS at `to` + 16 * lane (4 bytes: regs_copy_head), without a register in between.  All are
// called where every lane of the wavefront is on, which is what they leave.  (M0, which they and the index mode set, is a register that
// the compiler reserves: it sets it right before each use of its own and holds nothing in it over a statement.)
__device__ __forceinline__ void regs_copy(uint64_t from, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %1\n s_nop 0\n global_load_lds_dwordx4 %0, off" ::"v"(from), "s"(to) : "memory");
}
__device__ __forceinline__ void regs_copy_some(uint64_t from, uint32_t to, uint32_t lanes)  // the first 1 <= lanes < 64 of them
{
    asm volatile("s_mov_b32 m0, %1\n s_bfm_b64 exec, %2, 0\n global_load_lds_dwordx4 %0, off\n s_mov_b64 exec, -1" ::"v"(from), "s"(to),
                 "s"(lanes)
                 : "memory");
}
// The same from a uniform address + `offset`.  A scalar register that a vector instruction wrote (a lane read, a spill) may be an
// address five wait states later; the compiler counts none inside the statement, so they are all here.
__device__ __forceinline__ void regs_copy_list(uint64_t from, uint32_t offset, uint32_t to, uint32_t lanes)
{
    asm volatile("s_mov_b32 m0, %2\n s_nop 2\n s_bfm_b64 exec, %3, 0\n global_load_lds_dwordx4 %1, %0\n s_mov_b64 exec, -1" ::"s"(from), "v"(offset), "s"(to),
                 "s"(lanes)
                 : "memory");
}
__device__ __forceinline__ void regs_copy_head(uint64_t from, uint32_t offset, uint32_t to, uint32_t lanes)
{
    asm volatile("s_mov_b32 m0, %2\n s_nop 2\n s_bfm_b64 exec, %3, 0\n global_load_lds_dword %1, %0\n s_mov_b64 exec, -1" ::"s"(from), "v"(offset), "s"(to),
                 "s"(lanes)
                 : "memory");
}

// What a step takes from LDS before its copies and its list: the header of the step after next - head: first record and
// batches of the list; row[i]: row of copy i for this lane (`head_lane` says which of the copy's rows) - and the chunks of
// the present list.
template <int NR, int RPC, int CHUNKS, int CHUNK_BYTES>
__device__ __forceinline__ void regs_read(uint32_t at, uint32_t head_lane, uint32_t list_at, uint64_t& head, uint32_t (&row)[6], uint64_t (&chunk)[4])
{
    static_assert(NR == 3 || NR == 4 || NR == 6);
    static_assert(CHUNKS == 0 || CHUNKS == 1 || CHUNKS == 2 || CHUNKS == 4);
    const uint32_t rows_at = at + head_lane;
#define MAXK_ROW(I, J) "ds_read_b32 %[r" I "], %[ra] offset:8+" J "*%[s]\n"
#define MAXK_CHUNK(I) "ds_read_b64 %[c" I "], %[la] offset:" I "*%[cs]\n"
#define MAXK_READ(NR_TEXT, CH_TEXT)                                                                                            \
    asm volatile("ds_read_b64 %[h], %[at]\n" NR_TEXT CH_TEXT "s_waitcnt lgkmcnt(0)"                                             \
                 : [h] "=&v"(head), [r0] "=&v"(row[0]), [r1] "=&v"(row[1]), [r2] "=&v"(row[2]), [r3] "=&v"(row[3]), [r4] "=&v"(row[4]), \
                   [r5] "=&v"(row[5]), [c0] "=&v"(chunk[0]), [c1] "=&v"(chunk[1]), [c2] "=&v"(chunk[2]), [c3] "=&v"(chunk[3])    \
                 : [at] "v"(at), [ra] "v"(rows_at), [la] "v"(list_at), [s] "n"(4 * RPC), [cs] "n"(CHUNK_BYTES))
#define MAXK_ROWS3 MAXK_ROW("0", "0") MAXK_ROW("1", "1") MAXK_ROW("2", "2")
#define MAXK_ROWS4 MAXK_ROWS3 MAXK_ROW("3", "3")
#define MAXK_ROWS6 MAXK_ROWS4 MAXK_ROW("4", "4") MAXK_ROW("5", "5")
#define MAXK_CHUNKS1 MAXK_CHUNK("0")
#define MAXK_CHUNKS2 MAXK_CHUNKS1 MAXK_CHUNK("1")
#define MAXK_CHUNKS4 MAXK_CHUNKS2 MAXK_CHUNK("2") MAXK_CHUNK("3")
#define MAXK_READ_C(ROWS)                               \
    if constexpr (CHUNKS == 0) MAXK_READ(ROWS, "");      \
    else if constexpr (CHUNKS == 1) MAXK_READ(ROWS, MAXK_CHUNKS1); \
    else if constexpr (CHUNKS == 2) MAXK_READ(ROWS, MAXK_CHUNKS2); \
    else MAXK_READ(ROWS, MAXK_CHUNKS4);
    if constexpr (NR == 3) { MAXK_READ_C(MAXK_ROWS3) }
    else if constexpr (NR == 4) { MAXK_READ_C(MAXK_ROWS4) }
    else { MAXK_READ_C(MAXK_ROWS6) }
}
template <int N>
__device__ __forceinline__ void regs_wait_copies()  // all but the latest N copies of this wavefront have landed
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// G: destinations that share a register (64 / G lanes each); KR: registers a destination; PITCH: bytes of a row in LDS
template <int VT, int G, int KR, int PITCH>
__global__ __launch_bounds__(kRegsWaves* kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_regs_kernel(const RegsArgs a)
{
    constexpr RegsLayout L = regs_layout(PITCH);
    constexpr int LPR = PITCH <= 1024 ? PITCH / 16 : 64;           // lanes of a copy that share a row
    constexpr int RPC = 64 / LPR;                                  // rows of a copy
    constexpr int NR = L.rows / RPC, NC = PITCH <= 1024 ? NR : 2 * NR;  // copies for a wavefront's rows of a step
    constexpr int kCopies = NC + 2;  // copies of a step: rows, list, header
    constexpr int CHUNKS = 4 / G;  // 16 slots each: kRegsListRecords records
    constexpr int SLOTS = regs_slots(KR), VB = VT == MAXK_VALUE_F32 ? 4 : 2;
    constexpr uint32_t kTile = (uint32_t)(L.rows * kRegsWaves * PITCH), kList = 3 * kTile;
    constexpr uint32_t kHead = kList + 3 * kRegsWaves * kRegsListRecords * 16;
    static_assert(kHead + 4 * kRegsWaves * L.head * 4 <= 160 * 1024, "LDS");
    extern __shared__ __attribute__((aligned(16))) char regs_lds[];
    typedef __attribute__((address_space(3))) char lds_char;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)regs_lds;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const RegsUnit u = a.unit[blockIdx.x];
    const int g = lane / (64 / G), pos = lane % (64 / G);  // this lane's destinations and position(s): pos, pos + 64

    regs_v32 A0{}, A1{}, A2{}, C1{}, C2{}, C3{};
    regs_v16 A3{}, C0{};

    // ---- the columns of this wavefront's destinations ----
    const int32_t* const node = a.node + ((int64_t)u.set * kRegsWaves + wave) * (SLOTS * G);
    int32_t* const staged = reinterpret_cast<int32_t*>(regs_lds + wave * 2048);
    static_assert(SLOTS * G * 4 <= 2048, "a wavefront's nodes are staged in LDS");
    for (int i = lane; i < SLOTS * G; i += kWave) staged[i] = node[i];
    __builtin_amdgcn_wave_barrier();
    constexpr int NB = KR == 2 ? 8 : 16;
    static_assert(112 % (NB * KR) == 0);
    for (int r0 = 0; r0 < 112 / KR; r0 += NB) {
        uint32_t c[NB][KR];
        const auto load = [&](const auto* __restrict__ index) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int n = r0 + j < SLOTS ? staged[(r0 + j) * G + g] : -1;
#pragma unroll
                for (int h = 0; h < KR; ++h) {
                    const bool ok = n >= 0 && pos + 64 * h < a.k;
                    const uint32_t x = (uint32_t)index[ok ? (int64_t)n * a.k + (pos + 64 * h) : 0];
                    c[j][h] = ok ? x * VB : 0u;
                }
            }
        };
        if (a.index_bytes == 1) load(static_cast<const uint8_t*>(a.sp_index));
        else if (a.index_bytes == 2) load(static_cast<const uint16_t*>(a.sp_index));
        else load(static_cast<const int32_t*>(a.sp_index));
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
            for (int h = 0; h < KR; ++h) {
                // an entry's record holds the row's LDS address plus the number of its accumulator, which is taken off here
                const uint32_t x = c[j][h] - (uint32_t)((r0 + j) * KR);
                const int r = (r0 + j) * KR + h;
                asm volatile("s_set_gpr_idx_on %[r], 8\n v_mov_b32 v144, %[x]\n s_set_gpr_idx_off" : MAXK_REGS_FILE : [r] "s"(r), [x] "v"(x));
            }
        }
    }
    __syncthreads();

    // ---- the steps ----
    const int steps = u.end - u.begin;
    if (steps > 0) {
        const uint32_t row_bytes = a.row_bytes;
        const uint64_t dY = (uint64_t)(uintptr_t)a.dY;
        const uint64_t row0 = dY + (PITCH <= 1024 ? min((uint32_t)(lane % LPR) * 16u, row_bytes - 16u) : lane * 16u);
        const uint64_t row1 = dY + min(1024u + lane * 16u, row_bytes - 16u);  // second half of a long row
        const uint64_t rec0 = (uint64_t)(uintptr_t)a.rec;
        const uint32_t lane16 = lane * 16u;
        // Few vector registers are left beside the file and the list's; one spill in the loop would wait for the copies in flight.
        const auto lane4 = [&] {
            uint32_t x;
            asm volatile("v_lshrrev_b32 %0, 2, %1" : "=v"(x) : "v"(lane16));  // volatile: not kept over the loop
            return x;
        };
        constexpr uint32_t kListStride = kRegsWaves * kRegsListRecords * 16, kHeadStride = kRegsWaves * L.head * 4;
        const uint32_t list0 = lds0 + kList + wave * (kRegsListRecords * 16u), head0 = lds0 + kHead + wave * (L.head * 4u);
        const uint32_t my_rows = lds0 + wave * (L.rows * PITCH);
        const uint32_t head_lane = PITCH <= 1024 ? (uint32_t)(lane / LPR) * 4u : 0u;
        uint64_t head_at = (uint64_t)(uintptr_t)a.hdr + ((uint64_t)u.begin * kRegsWaves + wave) * (L.head * 4);

        // Copies of step s, from its header: its rows, its list, the header of step s + 2; returns the batches of its list.
        // Always the same number of copies, so that they can be counted; past the end of the unit they bring what nobody reads.
        uint32_t slot = 0;
        const auto issue = [&](int s, uint64_t head, const uint32_t (&row)[6]) -> uint32_t {
            const uint32_t first = __builtin_amdgcn_readfirstlane((uint32_t)head), n = __builtin_amdgcn_readfirstlane((uint32_t)(head >> 32));
            const uint32_t nb = n & 0xFFu, dst = my_rows + (n >> 8) * kTile;
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const uint64_t off = (uint64_t)row[i] * row_bytes;
                regs_copy(row0 + off, dst + i * (PITCH <= 1024 ? 1024 : PITCH));
                if constexpr (PITCH == 2048) regs_copy(row1 + off, dst + i * PITCH + 1024);
                if constexpr (PITCH == 1536) regs_copy_some(row1 + off, dst + i * PITCH + 1024, 32);
            }
            regs_copy_list(rec0 + (uint64_t)first * 16u, lane16, list0 + slot * kListStride, regs_copied(nb * (uint32_t)regs_batch_records(G, KR)));
            slot = slot == 2 ? 0 : slot + 1;
            regs_copy_head(head_at, lane4(), head0 + (uint32_t)((s + 2) & 3) * kHeadStride, L.head);
            head_at += (uint64_t)kHeadStride;
            return nb;
        };
        const auto header = [&](int s) { return head0 + (uint32_t)(s & 3) * kHeadStride; };
        uint64_t head, chunk[4];
        uint32_t row[6];
        regs_copy_head(head_at, lane4(), header(0), L.head);
        regs_copy_head(head_at + kHeadStride, lane4(), header(1), L.head);
        head_at += 2 * (uint64_t)kHeadStride;
        regs_wait_copies<0>();
        regs_read<NR, RPC, 0, 0>(header(0), head_lane, 0, head, row, chunk);
        uint32_t batches = issue(0, head, row);
        regs_read<NR, RPC, 0, 0>(header(1), head_lane, 0, head, row, chunk);
        uint32_t batches_next = issue(1, head, row);
        regs_wait_copies<kCopies>();
        __builtin_amdgcn_s_barrier();
        uint32_t list = 0;
        // constant address space: nothing writes it while the kernel runs, so it is read with scalar loads
        typedef const __attribute__((address_space(4))) RegsPart* const_part_ptr;
        const const_part_ptr part_list = (const_part_ptr)a.part;
        int part = u.part_begin, part_end = part < u.part_end ? part_list[part].end : -1;
        const uint32_t list_lane = list0 + (uint32_t)((lane % 16) * G + g) * 8u;
        for (int s = 0; s < steps; ++s) {
            // The buffers that step s + 2 fills were last read in step s - 1, which every wavefront has left.
            regs_read<NR, RPC, CHUNKS, 128 * G>(header(s + 2), head_lane, list_lane + list * kListStride, head, row, chunk);
            const uint32_t batches_after = issue(s + 2, head, row);
            list = list == 2 ? 0 : list + 1;
#define MAXK_REGS_FORMAT(LD, CV)                                                          \
    if constexpr (KR == 2) MAXK_REGS_LIST(BATCHES_P4, ADDR_W, FMA_W, LD, CV, "4");         \
    else if constexpr (G == 1) MAXK_REGS_LIST(BATCHES_Q4, ADDR_1, FMA_1, LD, CV, "4");     \
    else if constexpr (G == 2) MAXK_REGS_LIST(BATCHES_Q2, ADDR_2, FMA_2, LD, CV, "4");     \
    else MAXK_REGS_LIST(BATCHES_P1, ADDR_4, FMA_4, LD, CV, "2");
            if constexpr (VT == MAXK_VALUE_F32) { MAXK_REGS_FORMAT(LD_F32, CV_F32) }
            else if constexpr (VT == MAXK_VALUE_BF16) { MAXK_REGS_FORMAT(LD_16, CV_BF16) }
            else { MAXK_REGS_FORMAT(LD_16, CV_F16) }
#undef MAXK_REGS_FORMAT
            if (u.begin + s + 1 == part_end) {  // the sums of a part leave, and the next one starts from zero
                const int leaving = part_list[part].slots * KR;
                char* const out = reinterpret_cast<char*>(a.parts + (part_list[part].at + (int64_t)wave * leaving * kWave));
                const uint32_t at = lane4();
                for (int r0 = 0; r0 < leaving; r0 += 4) {
                    float x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        asm volatile("s_set_gpr_idx_on %[r], 1\n v_mov_b32 %[x], v32\n s_set_gpr_idx_mode 8\n v_mov_b32 v32, 0\n s_set_gpr_idx_off"
                                     : MAXK_REGS_FILE, [x] "=&v"(x[j]) : [r] "s"(r0 + j));
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (r0 + j < SLOTS * KR) *reinterpret_cast<float*>(out + (int64_t)(r0 + j) * (kWave * 4) + at) = x[j];
                }
                ++part;
                part_end = part < u.part_end ? part_list[part].end : -1;
            }
            batches = batches_next;
            batches_next = batches_after;
            regs_wait_copies<kCopies>();   // this wavefront's part of step s + 1 is in LDS ...
            __builtin_amdgcn_s_barrier();  // ... and everybody's
        }
        regs_wait_copies<0>();
        __builtin_amdgcn_s_barrier();
    }

    // ---- results of a set in one part ----
    if (u.part_begin < u.part_end) return;
    const int lane_ = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));  // again, so that it is not kept over the loop
    const int g_ = lane_ / (64 / G), pos_ = lane_ % (64 / G);
    for (int i = lane_; i < SLOTS * G; i += kWave) staged[i] = a.row[((int64_t)u.set * kRegsWaves + wave) * (SLOTS * G) + i];
    __builtin_amdgcn_wave_barrier();
    for (int r0 = 0; r0 < SLOTS; r0 += 8) {
        int n[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) n[j] = r0 + j < SLOTS ? staged[(r0 + j) * G + g_] : -1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
            for (int h = 0; h < KR; ++h) {
                float x;
                const int r = min((r0 + j) * KR + h, 111);
                asm volatile("s_set_gpr_idx_on %[r], 1\n v_mov_b32 %[x], v32\n s_set_gpr_idx_off" : MAXK_REGS_FILE, [x] "=v"(x) : [r] "s"(r));
                const int p = pos_ + 64 * h;
                if (n[j] >= 0 && p < a.k) (n[j] < a.N ? a.dXs : a.extra - a.N * a.k)[(int64_t)n[j] * a.k + p] = x;
            }
        }
    }
}

template <int VT, int G, int KR, int PITCH>
maxk_status launch_regs_t(const RegsArgs& a, int64_t n_units, hipStream_t s)
{
    constexpr int lds = 160 * 1024;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_regs_kernel<VT, G, KR, PITCH>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    MAXK_HIP_TRY(attr);
    hipLaunchKernelGGL((bwd_regs_kernel<VT, G, KR, PITCH>), dim3((unsigned)n_units), dim3(kRegsWaves * kWave), lds, s, a);
    MAXK_LAUNCH_CHECK();
    return MAXK_OK;
}

template <int VT, int G, int KR>
maxk_status launch_regs_p(int pitch, const RegsArgs& a, int64_t n_units, hipStream_t s)
{
    if constexpr (VT != MAXK_VALUE_F32 || KR == 1) {  // (256 bytes of fp32 are at most 64 columns, one register a destination)
        if (pitch == 256) return launch_regs_t<VT, G, KR, 256>(a, n_units, s);
    }
    return pitch == 512    ? launch_regs_t<VT, G, KR, 512>(a, n_units, s)
           : pitch == 1024 ? launch_regs_t<VT, G, KR, 1024>(a, n_units, s)
           : pitch == 1536 ? launch_regs_t<VT, G, KR, 1536>(a, n_units, s)
           : pitch == 2048 ? launch_regs_t<VT, G, KR, 2048>(a, n_units, s) : MAXK_UNSUPPORTED;
}

}  // namespace

template <int VT>
maxk_status launch_regs_format(const RegsSet& T, const void* dY, const void* sp_index, int index_bytes, int64_t N, int dim, int k, float* dXs,
                               hipStream_t s)
{
    const RegsArgs a = {dY, sp_index, dXs, T.d_rec, T.d_hdr, T.d_node, T.d_row, T.d_extra, N, T.d_unit, T.d_part, T.d_parts, (uint32_t)dim * (VT == MAXK_VALUE_F32 ? 4u : 2u), k, index_bytes};
    const int pitch = T.shape.pitch;
    return T.shape.kr == 2       ? launch_regs_p<VT, 1, 2>(pitch, a, T.n_units, s)
           : T.shape.groups == 1 ? launch_regs_p<VT, 1, 1>(pitch, a, T.n_units, s)
           : T.shape.groups == 2 ? launch_regs_p<VT, 2, 1>(pitch, a, T.n_units, s)
                                 : launch_regs_p<VT, 4, 1>(pitch, a, T.n_units, s);
}

}  // namespace maxk
