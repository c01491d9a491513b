// Action calls on energy tables that are already on the device, for
// integrators that apply many exponentials exp(-i t (alpha H_P + beta sum_j X_j))
// with the same couplings (defined in qw_action.hip).
#pragma once

#include "qw_device.h"
#include "qwexp.h"

#include <vector>

namespace qw {

// Device tables of one (h, J) set and, for an action call, the factor alpha by
// which the energies are scaled.
struct Prepared {
    EnergyTables T;
    bool have_q;      // T's pair table has been built
    double escale;
};

// Puts (h, J) into the workspace (qw_workspace_bytes layout), builds the pair
// table where the action of that size reads one, and returns min / max of E
// over all 2^n states (one read-back, none up to 13 qubits).
template <typename R>
qw_status prepare_energy(int n, const double *h, const double *J, void *workspace, size_t ws_bytes, void *stream,
                         EnergyTables *T, bool *have_q, double *emin, double *emax);

// psi_out = exp(-i t (alpha H_P + beta sum_j X_j)) psi_in with the prepared
// tables; the shift and bound follow from alpha, [emin, emax] and beta without
// a read-back, and the norm monitor stays off.
template <typename R>
qw_status scaled_action(int n, const double *h, const double *J, const EnergyTables &T, bool have_q, double alpha,
                        double emin, double emax, double beta, double t, const void *psi_in, void *psi_out, double tol,
                        void *workspace, size_t ws_bytes, void *stream, qw_info *info);

// Whether exponentials of n qubits can be applied several to a launch on this
// stream, and whether such a launch can be recorded into a graph.
template <typename R> bool chain_fits(int n, void *stream);
template <typename R> bool chain_captures(int n);

// Up to CHAIN_ITEMS exponentials exp(-i t (alpha H_P + beta sum_j X_j)), the
// first first, in one launch (psi_out may be psi_in); adds their degrees to
// *terms.  *refused: the launch was refused, nothing has been applied.
struct ChainItem {
    double alpha, beta, t, tol;
};
static constexpr int CHAIN_ITEMS = 32;
template <typename R>
qw_status scaled_chain(int n, const EnergyTables &T, double emin, double emax, const std::vector<ChainItem> &items,
                       const void *psi_in, void *psi_out, void *workspace, size_t ws_bytes, void *stream,
                       long long *terms, bool *refused);

}  // namespace qw
