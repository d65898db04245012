// Phases of the cycle counters of profiling builds (-DQPK_PHASE_TIMING): one
// list gives the kernels' indices and the names they are reported under.
#pragma once

#define QPK_PHASE_LIST(X)                                                      \
  X(PH_INIT, "init")                                                           \
  X(PH_RESID, "resid")                                                         \
  X(PH_PART, "part")                                                           \
  X(PH_ASM, "asm")                                                             \
  X(PH_FACT, "fact")                                                           \
  X(PH_RHS, "rhs")                                                             \
  X(PH_SOLVE, "solve")                                                         \
  X(PH_REFINE, "refine")                                                       \
  X(PH_RECOVER, "recover")                                                     \
  X(PH_STEP, "step")                                                           \
  X(PH_BWD, "bwd")                                                             \
  X(PH_OUT, "out")                                                             \
  X(PH_ASM_BORDER, "asm_border")                                               \
  X(PH_ASM_DIAG, "asm_diag")                                                   \
  X(PH_FACT_UPDATE, "fact_update")                                             \
  X(PH_FACT_ELIM, "fact_elim")                                                 \
  X(PH_MATVEC, "matvec")                                                       \
  X(PH_KAPPA, "kappa")                                                         \
  X(PH_AFFINE, "affine")                                                       \
  X(PH_REFINE_APPLY, "refine_apply")

#define QPK_PHASE_INDEX(index, name) index,
#define QPK_PHASE_NAME(index, name) name,

// Counters of a QP: one per phase, and the previous mark's clock in the last.
enum Phase { QPK_PHASE_LIST(QPK_PHASE_INDEX) PH_COUNT, PH_N = 32 };
static_assert(PH_COUNT < PH_N, "a counter per phase and one for the clock");

static const char *const kPhaseNames[] = {QPK_PHASE_LIST(QPK_PHASE_NAME)};
static_assert(sizeof(kPhaseNames) / sizeof(kPhaseNames[0]) == PH_COUNT, "a name per phase");
