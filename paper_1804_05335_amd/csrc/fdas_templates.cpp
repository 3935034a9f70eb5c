// Host side of the template math (see fdas_response.hpp).
#include <complex>

#include "fdas_internal.h"
#include "fdas_response.hpp"

namespace fdas {

std::complex<double> response(double q, double z)
{
    const cplx64 r = response64(q, z);
    return {r.re, r.im};
}

}  // namespace fdas
