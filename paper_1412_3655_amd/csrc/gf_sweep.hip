// gf_sweep.hip -- the single-lattice half-sweep launchers of libgf on gfx950:
// Landau gauge here (K over all 4 directions, Eq. localfunctional of
// arXiv:1412.3655); the Coulomb instantiation of the same kernel is compiled
// in gf_sweep_coulomb.hip and reached through the gauge argument, the
// estimating sweeps in gf_sweep_est.hip / gf_sweep_coulomb_est.hip.
#include "gf_sweep_impl.h"

namespace gf {

bool sweep_config_valid(const SweepConfig& c)
{
    const bool tps_ok = c.tps == 1 || c.tps == 2 || c.tps == 4 || c.tps == 8;
    const bool blk_ok = c.block == 64 || c.block == 128 || c.block == 256 || c.block == 512;
    const bool nt_ok = c.nt == 0 || ((c.nt == 1 || c.nt == 2) && c.tps <= 4 && c.block <= 256);
    const bool minw_ok = c.minw == 0 || (c.minw == 2 && c.tps == 1);
    // one lane per site needs more than the 256 registers a 512-thread block allows
    return tps_ok && blk_ok && nt_ok && minw_ok && !(c.tps == 1 && c.block == 512);
}

// Every configuration gives the same links, so only time decides.  The lines are
// where the tuner's tables over 4^4 .. 48^3x96 in every precision and storage
// cross; the rule's choice is within 3 % of the best of each table on average
// (4 lanes, 256 threads, plain accesses everywhere: 19 %).
//   - Few sites: a half-sweep is one round of waves and costs its latency, so a
//     site's work is spread over lanes and the blocks over compute units (8^4
//     float64, us per sweep: 4 lanes in blocks of 64 9.8, of 256 11.9; 8-real
//     links, whose decode dominates, 8 lanes 10.6, 4 lanes 11.4).
//   - A field that fits the 8 L2s (32 MiB, somewhat more as reads leave no dirty
//     lines): non-temporal.  With plain stores the half-sweep ends by flushing
//     the dirty field from L2, where non-temporal ones are long written through:
//     16^4 float32 24.8 -> 12.0, SU(2) 16^3x32 float64 27.6 -> 10.9.  Beyond, plain
//     loads find part of the previous half-sweep in the Infinity Cache (24^4
//     float64 82 plain, 102 non-temporal).
//   - Otherwise 2 lanes: enough waves per SIMD to hide the loads without
//     repeating the subgroup algebra in 4 (32^4 float32 8-real 99 against 126);
//     one lane for the heat bath, which samples in every lane, unless the
//     lattice leaves SIMDs idle (16^4 float32: 2 lanes 31, 1 lane 35; 32^4: 165
//     at 1 lane, 194 at 2), in blocks of 64, which spread the few waves of a
//     middling lattice evenly (16^3x32 float32 37 us, blocks of 128 45; 24^3x48
//     8 reals 107, 113).
SweepConfig default_sweep_config(const Geom& g, bool f64, int reals, bool heat_bath)
{
    const uint64_t bytes = (uint64_t)g.vh * 8 * (uint64_t)reals * (f64 ? 8 : 4);
    constexpr uint32_t kTiny = 5120, kSmall = 12288, kMedium = 40960;
    if (reals == 4) {
        const bool nt = g.vh > kTiny && bytes <= (32u << 20);
        return SweepConfig{1, g.vh <= kSmall ? 64 : 256, nt ? 1 : 0, 0};
    }
    const bool nt = bytes <= (48u << 20);
    if (g.vh <= kTiny) return SweepConfig{reals == 8 || heat_bath ? 8 : 4, 64, 0, 0};
    if (g.vh <= kSmall) return SweepConfig{reals == 8 || heat_bath ? 4 : 2, 64, 1, 0};
    if (heat_bath && g.vh > kMedium) return SweepConfig{1, 64, nt ? 1 : 0, 0};
    if (nt) return SweepConfig{2, 256, 1, 0};
    return SweepConfig{2, reals == 8 ? 64 : 256, 0, 0};
}

hipError_t launch_or_half_sweep(const LinkField<double>& f, const Geom& g, int parity, const OrOmega& om, int mode,
                                const SweepConfig& cfg, hipStream_t st, int gauge, double* est)
{
    if (gauge == GAUGE_COULOMB) return launch_or_half_sweep_coulomb(f, g, parity, om, mode, cfg, st, est);
    if (est) return launch_or_half_sweep_est(f, g, parity, om, mode, cfg, st, est);
    return sweep_impl::or_half_sweep<NDIR_LANDAU, false>(f, g, parity, om, mode, cfg, st, nullptr);
}

hipError_t launch_or_half_sweep(const LinkField<float>& f, const Geom& g, int parity, const OrOmega& om, int mode,
                                const SweepConfig& cfg, const GField& gacc, hipStream_t st, int gauge, double* est)
{
    if (gauge == GAUGE_COULOMB)
        return launch_or_half_sweep_coulomb(f, g, parity, om, mode, cfg, gacc, st, est);
    if (est) return launch_or_half_sweep_est(f, g, parity, om, mode, cfg, gacc, st, est);
    return sweep_impl::or_half_sweep<NDIR_LANDAU, false>(f, g, parity, om, mode, cfg, gacc, st, nullptr);
}

uint32_t sweep_blocks(const Geom& g, const SweepConfig& cfg)
{
    return sweep_impl::sweep_grid(g, cfg);
}

hipError_t launch_hb_half_sweep(const LinkField<double>& f, const Geom& g, int parity, double T, uint64_t seed,
                                uint32_t sweep, const SweepConfig& cfg, hipStream_t st, int gauge)
{
    if (gauge == GAUGE_COULOMB) return launch_hb_half_sweep_coulomb(f, g, parity, T, seed, sweep, cfg, st);
    return sweep_impl::hb_half_sweep<NDIR_LANDAU>(f, g, parity, T, seed, sweep, cfg, st);
}

hipError_t launch_hb_half_sweep(const LinkField<float>& f, const Geom& g, int parity, float T, uint64_t seed,
                                uint32_t sweep, const SweepConfig& cfg, const GField& gacc, hipStream_t st, int gauge)
{
    if (gauge == GAUGE_COULOMB) return launch_hb_half_sweep_coulomb(f, g, parity, T, seed, sweep, cfg, gacc, st);
    return sweep_impl::hb_half_sweep<NDIR_LANDAU>(f, g, parity, T, seed, sweep, cfg, gacc, st);
}

}  // namespace gf
