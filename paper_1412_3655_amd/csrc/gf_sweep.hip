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
// where tables of all configurations over 41 lattices from 4^4 to 48^3x96, in every
// precision and storage and both gauges, cross; the rule's choice is within 2 % of
// the best of a table on average and within 11 % at worst.  (Below in us per sweep.)
//   - One round: a half-sweep of few sites costs the latency of a wave, so a site
//     goes to as many lanes as leave at most one wave on each of the 1024 SIMDs:
//     kOneRound sites per colour at one lane, half of that at two.  8 reals and the
//     heat bath, whose decode or sampling is long, follow this to 8 lanes (heat
//     bath of float64 12 reals: 7200 sites at 8 lanes 34.0, at 4 35.4; 32768 at 2
//     42, at 1 48; 40960 at 1 49, at 2 69).  Sweeps of 12 reals repeat their algebra in
//     every lane and change earlier (float64, 5120 sites: 2 lanes 10.8, 4 lanes
//     12.6), and just below one lane's round more waves hide what a single one
//     cannot (46080 sites: float64 12 reals, 2 lanes 21, 1 23; 8 reals, 4 lanes
//     24, 1 27; float32 12 reals, 2 lanes 16.4, 1 18.5; 8 reals 20.7 and 22.0).
//   - A field that the 8 L2s hold: non-temporal.  With plain stores the half-sweep
//     ends by flushing the dirty field from L2, where non-temporal ones are long
//     written through: 16^4 float32 24 -> 13, SU(2) 16^3x32 float64 27.6 -> 10.9.
//     Beyond, plain loads find part of the previous half-sweep in the Infinity
//     Cache.  The tables cross at 48 MiB for float64 (58 MiB: 42 plain, 47
//     non-temporal) and 8 reals, at 30 MiB for float32 in 12 reals (46 MiB: plain
//     30.3, non-temporal at two lanes 37.6), at 24 for SU(2) (28 MiB: 20.1 and
//     22.3; its heat bath at 32).  Half a MiB has no time to flush: plain (SU(2),
//     864 sites: 6.3 and 7.0).
//   - Beyond, 2 lanes hide the loads without repeating the algebra in 4, but one is
//     enough in float32 12 reals (32^4 118, 2 lanes 120) and in the heat bath (32^4
//     142 and 170), there in blocks of 64, which spread the waves evenly.
//   - Float32 links in 8 reals that the 256 MB Infinity Cache no longer holds (with
//     g, if tracked) are non-temporal again (32^3x64 mixed 216, plain 243), and at
//     one lane when they are far beyond (48^3x96 984, 2 lanes plain 1067).  Without
//     g, between the two, one lane with plain accesses is 3 to 6 % ahead.
SweepConfig default_sweep_config(const Geom& g, bool f64, int reals, bool heat_bath, bool tracked)
{
    constexpr uint32_t kOneRound = 65536;
    constexpr uint64_t MiB = 1u << 20;
    const uint64_t bytes = (uint64_t)g.vh * 8 * (uint64_t)reals * (f64 ? 8 : 4);
    const uint32_t n = g.vh;
    if (reals == 4) {
        if (bytes <= MiB / 2) return SweepConfig{1, 64, 0, 0};
        if (bytes > (heat_bath ? 32 : 24) * MiB) return SweepConfig{1, 256, 0, 0};
        if (n <= (heat_bath ? kOneRound / 2 : kOneRound / 8)) return SweepConfig{1, 64, 1, 0};
        if (heat_bath) return SweepConfig{1, 256, 1, 0};
        if (n <= kOneRound / 2) return SweepConfig{1, 128, 1, 0};
        if (n <= kOneRound) return SweepConfig{1, 256, 1, 0};
        if (f64) return SweepConfig{1, 128, 1, 0};
        return SweepConfig{1, n <= 2 * kOneRound ? 512 : 256, 1, 0};
    }
    const bool in_l2 = bytes <= 48 * MiB;
    if (reals == 8 || heat_bath) {
        if (n <= (heat_bath || !f64 ? kOneRound / 8 : 6144)) return SweepConfig{8, 64, 0, 0};
        if (n <= kOneRound / 4) return SweepConfig{4, 256, 1, 0};
        if (n <= kOneRound / 2) return SweepConfig{2, 256, 1, 0};
        if (heat_bath) return SweepConfig{1, 64, in_l2 ? 1 : 0, 0};
        if (f64) {
            if (n <= kOneRound / 4 * 3) return SweepConfig{4, 64, 1, 0};
            if (n <= kOneRound) return SweepConfig{1, 256, 1, 0};
            return in_l2 ? SweepConfig{2, 256, 1, 0} : SweepConfig{2, 64, 0, 0};
        }
        // 1 lane up to two thirds of its round, and again towards the end of its second
        if (n <= kOneRound / 3 * 2 || (n > kOneRound / 2 * 3 && n <= 2 * kOneRound)) return SweepConfig{1, 256, 1, 0};
        const uint64_t all = bytes + (tracked ? (uint64_t)n * 2 * 48 : 0);
        if (all > 352 * MiB) return SweepConfig{1, 64, 1, 0};
        if (all > 256 * MiB) return tracked ? SweepConfig{2, 64, 1, 0} : SweepConfig{1, 64, 0, 0};
        return SweepConfig{2, 64, in_l2 ? 1 : 0, 0};
    }
    if (n <= (f64 ? 2560 : kOneRound / 16)) return SweepConfig{4, 64, 0, 0};
    if (n <= kOneRound / 8) return f64 ? SweepConfig{2, 64, 1, 0} : SweepConfig{4, 128, 1, 0};
    if (n <= kOneRound / 4) return SweepConfig{2, 128, 1, 0};
    if (n <= kOneRound / 2) return SweepConfig{2, 256, 1, 0};
    if (f64) {
        if (n <= kOneRound / 4 * 3) return SweepConfig{2, 64, 1, 0};
        return n <= kOneRound ? SweepConfig{1, 64, 1, 0} : SweepConfig{2, 256, 0, 0};
    }
    if (n <= kOneRound / 3 * 2) return SweepConfig{1, 256, 1, 0};
    if (n <= kOneRound / 8 * 7) return SweepConfig{2, 64, 1, 0};
    return n <= kOneRound / 4 * 5 ? SweepConfig{2, 128, 1, 0} : SweepConfig{1, 256, 0, 0};
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
