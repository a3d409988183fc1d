/*
 * gbp_test_hooks.h -- entry points of libgbp that exist for tests only.  They
 * reach states that ordinary use meets rarely or never, so that the code paths
 * for those states can be tested.  Not part of the solver interface (gbp.h).
 */
#ifndef GBP_TEST_HOOKS_H
#define GBP_TEST_HOOKS_H

#include "gbp.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * gbp_plan_set_stamp_base -- sets the base of the forward's queue stamps (each
 * relaxation round marks queued vertices with the base plus its round index; the
 * base restarts from 1, clearing every mark, once it exceeds 2^30).  The restart
 * otherwise comes after some ten million solves on one plan.  Synchronises the
 * device.  Errors: GBP_ERR_ARG for stamp < 1, GBP_ERR_HIP.
 */
int gbp_plan_set_stamp_base(gbp_plan plan, int stamp);

/*
 * gbp_plan_set_team, gbp_tri_plan_set_team -- bounds on the teams of blocks that run a
 * solve's rounds, the adjoint's levels and its sweeps in one launch (0: none): the
 * blocks that found a team (the others join at the ends of rounds) and its blocks in
 * all.  Otherwise a small or growing team needs a device that other work fills.
 * Results do not depend on them.  Errors: GBP_ERR_ARG for negative bounds.
 */
int gbp_plan_set_team(gbp_plan plan, int founders, int most);
int gbp_tri_plan_set_team(gbp_tri_plan plan, int founders, int most);

/*
 * gbp_plan_team, gbp_tri_plan_team -- blocks that founded the last launch's team and
 * its blocks at the end.  Synchronises the device.  Errors: GBP_ERR_HIP.
 */
int gbp_plan_team(gbp_plan plan, int *founders, int *members);
int gbp_tri_plan_team(gbp_tri_plan plan, int *founders, int *members);

#ifdef __cplusplus
}
#endif
#endif /* GBP_TEST_HOOKS_H */
