/*
 * eselbm_rollout.h -- sequences of calls of eselbm.h as a differentiable
 * rollout makes them, for callers whose own loop costs more than the kernels
 * it launches (a small lattice steps in a few microseconds).  Each function
 * makes the calls named here, in this order and with these arguments, and
 * returns the first status that is not ESELBM_OK; the arguments of all of
 * them are checked before the first is made.
 */
#ifndef ESELBM_ROLLOUT_H
#define ESELBM_ROLLOUT_H

#include "eselbm.h"

#ifdef __cplusplus
extern "C" {
#endif

/* n >= 1 steps f -> states[0] -> ... -> states[n - 1]: for every k
 * eselbm_step(previous, states[k], 1, tau).  With uvs (NULL, or n device
 * velocity fields), uvs[k] is registered for step k (eselbm_set_velocity_field)
 * and none afterwards; with loss_dev as well, every step is followed by
 * eselbm_dissipation_loss_uv(uvs[k], loss_dev, NULL, NULL, weight, NULL).
 * Consecutive entries of states differ; f is not written unless it is one of
 * them. */
eselbm_status eselbm_rollout_steps(eselbm_handle h, const void *f, void *const *states, float *const *uvs, int n,
                                   double tau, double *loss_dev, double weight, void *stream);

/* n >= 1 adjoint steps, the state before step k being states[k] (in the order
 * of application, the newest first): lam -> other -> lam ..., the last result
 * in other when n is odd and in lam when it is even.  With uvs (NULL, or n
 * entries) and uvs[k] not NULL, step k is eselbm_adjoint_step_diss with that
 * velocity field and weight, else eselbm_adjoint_step without a seed. */
eselbm_status eselbm_rollout_adjoints(eselbm_handle h, const void *const *states, const float *const *uvs, int n,
                                      double weight, void *lam, void *other, double tau, void *force_grad,
                                      void *stream);

#ifdef __cplusplus
}
#endif

#endif /* ESELBM_ROLLOUT_H */
