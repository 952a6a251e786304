// Resident CG (resident.hip): plan and entry points.
#pragma once
#include "pc_ctx.h"

namespace pc {

struct SpmvArgs;

// Dynamic LDS of a resident workgroup: the direction's window (16 bytes a
// row) and the vectors it keeps there, of the 160 KiB a compute unit has.
constexpr int RES_LDS = 152 * 1024;
// Window rows that fit, for vectors of 4 or 8 bytes a value.
int resident_win_max(const Ctx *ctx);

pc_status resident_plan(Ctx *ctx);
void resident_free(Ctx *ctx);
pc_status resident_windows(Ctx *ctx, int *inst_win, bool *fits, hipStream_t s);
bool resident_fits(const Ctx *ctx);
// Run every unfinished instance whose window fits for up to max_iters
// iterations from its state at parity ctx->cg_par (left unchanged).  *taken:
// false when the runtime refused a launch; instances of the rounds before it run,
// the others' states are as they were.
template <typename TB>
pc_status resident_launch(Ctx *ctx, const SpmvArgs &M, int max_iters, bool *taken, hipStream_t s);

}  // namespace pc
