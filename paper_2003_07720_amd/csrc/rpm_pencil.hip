// Instantiations of the fixed-length pencil passes (rpm_pencil.h): every length
// of RPM_PENCIL_LENGTHS, or those of one group (the build compiles the groups
// side by side).
#include "rpm_pencil.h"

#include <type_traits>

namespace rpm {

template <typename T, int N>
void Pencil<T, N>::y_pass(int dir, int comps, const cx<T>* in, cx<T>* out, const Geo& g, const cx<T>* tw,
                          const int* done, hipStream_t s)
{
    const int nzt = (g.nz + rows() - 1) / rows(), grid = comps * g.nh * nzt;
    constexpr int NT = tile_threads<T, N>();
    const PyArgs<T> a{in, out, tw, done, g.nh, g.nz, nzt};
    if (dir < 0) k_py<T, N, -1><<<grid, NT, 0, s>>>(a);
    else k_py<T, N, +1><<<grid, NT, 0, s>>>(a);
}

template <typename T, int N>
void Pencil<T, N>::x_forward(bool pol, const T* xin, const uint8_t* phase, const double* lame, int use_ref,
                             double lam0, double mu0, cx<T>* S1, double* part_mean, const Geo& g, const cx<T>* tw,
                             const int* done, hipStream_t s)
{
    const int nyt = (g.ny + rows() - 1) / rows(), nt = g.nz * nyt;
    constexpr int NT = tile_threads<T, N>();
    const PxfArgs<T> a{xin, phase, lame, S1, part_mean, tw, done, lam0, mu0, use_ref, g.nph, g.ny, g.nz, nt, nyt};
    if (pol) k_pxf<T, N, 6><<<x_grid(nt, 6), NT, 0, s>>>(a);
    else k_pxf<T, N, 3><<<x_grid(nt, 3), NT, 0, s>>>(a);
}

template <typename T, int N>
void Pencil<T, N>::x_inverse(bool pol, const cx<T>* S1, const T* eps, T* out, int out_mode, const T* shift,
                             double* part_inc, const Geo& g, const cx<T>* tw, const uint8_t* phase,
                             const double* lame, double lam0, double mu0, double beta, const int* done,
                             hipStream_t s)
{
    const int nyt = (g.ny + rows() - 1) / rows(), nt = g.nz * nyt;
    constexpr int NT = tile_threads<T, N>();
    if (pol)
        k_pxi_pol<T, N><<<nt, pol_groups<T, N>() * NT, 0, s>>>(PxpArgs<T>{
            S1, eps, out, shift, part_inc, tw, phase, lame, done, lam0, mu0, beta, g.ny, g.nz, nyt});
    else
        k_pxi<T, N><<<x_grid(nt, 3), NT, 0, s>>>(
            PxiArgs<T>{S1, eps, out, shift, part_inc, tw, done, out_mode, g.ny, g.nz, nt, nyt});
}

template <typename T, int N>
void Pencil<T, N>::gamma(bool pol, cx<T>* S, const Geo& g, const cx<T>* tw, double lam0, double mu0, double alpha,
                         double beta, int dc_mode, const double* E, const double* part_mean, int n_mean,
                         double* part_err, DevState* st, const int* done, hipStream_t s)
{
    const int npen = g.two_d ? g.nh : g.ny * g.nh;
    PgArgs<T> a{S,   tw,  E,    part_mean,    part_err, st,   done,
                lam0, mu0, {g.kh[0], g.kh[1], g.kh[2]}, g.nx, g.ny, g.nz, dc_mode == DC_MEAN ? n_mean : 0};
    if (pol) {
        a.c[0] = alpha;
        a.c[1] = beta;
    }
    auto launch = [&](auto p, auto w) {
        constexpr bool POL = decltype(p)::value, W = decltype(w)::value;
        k_pg<T, N, POL, W><<<gamma_blocks(POL, npen), GCfg<T, N, POL, W>::NT, 0, s>>>(a);
    };
    using std::false_type, std::true_type;
    if (pol) {
        if constexpr (pol_gamma<T, N>()) launch(true_type(), true_type());
    } else if constexpr (always_wide<T, N>(false)) launch(false_type(), true_type());
    else if (gamma_wide<T, N>(false, npen)) launch(false_type(), true_type());
    else launch(false_type(), false_type());
}

#define RPM_INST(N)              \
    template struct Pencil<float, N>; \
    template struct Pencil<double, N>;

#if !defined(RPM_PENCIL_GROUP)
RPM_PENCIL_LENGTHS(RPM_INST)
#elif RPM_PENCIL_GROUP == 0
RPM_INST(16) RPM_INST(64) RPM_INST(256)
#elif RPM_PENCIL_GROUP == 1
RPM_INST(18) RPM_INST(72) RPM_INST(128)
#elif RPM_PENCIL_GROUP == 2
RPM_INST(24) RPM_INST(81) RPM_INST(192)
#elif RPM_PENCIL_GROUP == 3
RPM_INST(27) RPM_INST(48) RPM_INST(162)
#elif RPM_PENCIL_GROUP == 4
RPM_INST(32) RPM_INST(54) RPM_INST(144)
#else
RPM_INST(36) RPM_INST(96) RPM_INST(108)
#endif

}  // namespace rpm
