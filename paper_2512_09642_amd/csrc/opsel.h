// Device operator functors (common.h) built from the library's device copy of
// an operator, in either precision.
#pragma once

#include "ell_rule.h"
#include "launch.h"

namespace sstep {

template <typename T>
inline OpPoisson7<T> make_poisson(const OpDev &op)
{
    return OpPoisson7<T>{op.g, op.precond ? T(1) / T(6) : T(1)};
}

template <typename T>
inline OpPoisson27<T> make_poisson27(const OpDev &op)
{
    return OpPoisson27<T>{op.g, op.precond ? T(1) / T(26) : T(1)};
}

template <typename T>
struct Ops;
template <>
struct Ops<double> {
    static OpFaces7<double> faces(const OpDev &op) { return {op.g, op.kx, op.ky, op.kz, op.precond}; }
    static OpCsr<double> csr(const OpDev &op) { return {op.rp, op.ci, op.val, op.invd}; }
    template <bool KEEP>
    static OpEll<double, KEEP> ell(const OpDev &op)
    {
        return {op.ell_slice, op.ell_col, op.ell_val, op.ell_dofs, op.ell_dmask, nullptr, static_cast<int32_t>(op.n),
                op.precond};
    }
};
template <>
struct Ops<float> {
    static OpFaces7<float> faces(const OpDev &op) { return {op.g, op.kx32, op.ky32, op.kz32, op.precond}; }
    static OpCsr<float> csr(const OpDev &op) { return {op.rp, op.ci, op.val32, op.invd32}; }
    template <bool KEEP>
    static OpEll<float, KEEP> ell(const OpDev &op)
    {
        return {op.ell_slice, op.ell_col, op.ell_val32, op.ell_dofs, op.ell_dmask, op.invd32,
                static_cast<int32_t>(op.n), op.precond};
    }
};

inline bool ell_keep(const OpDev &op, int elem) { return ell_keep_pays(op.ell_values, op.ell_span, elem); }

}  // namespace sstep
