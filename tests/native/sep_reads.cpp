// Host check of the separable kernels' record reads: for plans of many shapes,
// every record that a thread of k_step_sep2/3 or k_adjoint_sep2/3 reads, with or
// without weight, lies in the instance's reachable box (where the slope pass
// writes records), at any drift within the plan's bound.  Built with the plan
// builder's own source, so that its lists are seen as the kernels get them.
#include "fk_host.cpp"

#include <cstdlib>

namespace {

struct Axis1 { double lo, h; int n, periodic; };

long long checked = 0, bad = 0, sep_nodes = 0, plans = 0;

// wrap_index of the kernels
int wrap(int i, int n, bool per)
{
    if (per) return i < 0 ? i + n - 1 : (i > n - 1 ? i - (n - 1) : i);
    return i < 0 ? 0 : (i > n - 1 ? n - 1 : i);
}

// columns read past a footprint's first node, as the kernels unroll them
int columns(int d, int L, int a, const int *own)
{
    const int o = std::min(own[a], L);
    if (d == 2) return a == 1 ? (L > 6 || o > 3 ? L : 3) : o;
    return a == 2 || L <= 4 ? L : o;
}

void check_list(const fk_plan *p, const std::vector<int> &nodes, const std::vector<fk::WorkItem> &work,
                const int *off, const int *cnt, const char *what)
{
    for (int c = 0; c < fk::kBoxClasses; ++c)
        for (int t = off[c]; t < off[c] + cnt[c]; ++t) {
            const fk::WorkItem &it = work[t];
            const fk::DevInst &I = p->inst[it.inst];
            const fk_problem &pr = p->probs[it.inst];
            const int L = fk::box_len(p->d, c);
            for (int u = 0; u < it.count; ++u) {
                int r = nodes[it.first + u], idx[3];
                for (int a = p->d - 1; a >= 0; --a) { idx[a] = r % I.n[a]; r /= I.n[a]; }
                ++sep_nodes;
                for (int a = 0; a < p->d; ++a) {
                    const double B = drift_bound(pr, a) * pr.dt / I.step[a];
                    for (double b : {-B, 0.0, B}) {
                        const int o = idx[a] + (int)std::floor(std::fma(p->gh_a[0], I.S * I.inv_h[a], b));
                        for (int k = 0; k < columns(p->d, L, a, I.sep_l); ++k) {
                            const int m = wrap(o + k, I.n[a], I.periodic[a] != 0);
                            ++checked;
                            if (m >= I.blo[a] && m < I.blo[a] + I.blen[a]) continue;
                            if (bad++ < 5)
                                printf("%s: axis %d of %d: node %d reads %d, records at %d .. %d (class %d, footprint %d, n %d)\n",
                                       what, a, p->d, idx[a], m, I.blo[a], I.blo[a] + I.blen[a] - 1, L,
                                       I.sep_l[a], I.n[a]);
                        }
                    }
                }
            }
        }
}

void check(int d, const Axis1 *ax, double drift, double D, double dt, int q, bool ball, double radius, int f32)
{
    std::vector<std::vector<double>> nodes(d);
    fk_problem pr{};
    pr.d = d;
    for (int a = 0; a < d; ++a) {
        for (int k = 0; k < ax[a].n; ++k) nodes[a].push_back(k * ax[a].h + ax[a].lo);
        pr.ax[a] = {ax[a].n, nodes[a].data(), ax[a].periodic};
        pr.center[a] = ax[a].lo + 0.4 * (ax[a].n - 1) * ax[a].h;
        pr.coef[a] = drift;
    }
    pr.coef_kind = FK_COEF_CONST;
    pr.D = D;
    pr.region_kind = ball ? FK_REGION_BALL : FK_REGION_BOX;
    pr.radius = radius;
    pr.gh_q = q;
    pr.dt = dt;
    pr.n_steps = 2;
    fk_options o{};
    o.precision = f32 ? FK_PREC_F32 : FK_PREC_F64;
    o.ckpt_every = 1;
    o.step_kernel = 4;
    fk_plan *p = nullptr;
    if (fk_plan_create(&pr, 1, &o, &p) != FK_OK) {
        printf("plan refused: %s\n", fk_last_error());
        ++bad;
        return;
    }
    p->probs[0] = pr;   // (the plan's copy drops the caller's arrays)
    ++plans;
    check_list(p, p->box_nodes, p->box_work, p->box_work_off, p->n_box_work, "step");
    check_list(p, p->adj.box_nodes, p->adj.box_work, p->adj.box_work_off, p->adj.n_box_work, "transposed step");
    fk_plan_destroy(p);
}

}  // namespace

int main()
{
    unsigned long long s = 12345;
    auto rnd = [&] {   // uniform in [0, 1)
        s = s * 6364136223846793005ull + 1442695040888963407ull;
        return (double)(s >> 11) / 9007199254740992.0;
    };
    for (int t = 0; t < 300; ++t) {
        const int d = t % 3 == 2 ? 3 : 2;
        Axis1 ax[3];
        const double h = 0.01, dt = 1e-3;
        const bool ball = t % 2 == 0 && t % 5 != 4;   // no ball on periodic axes
        double span = 1e9;
        for (int a = 0; a < d; ++a) {
            ax[a].h = h * std::pow(8.0, rnd());   // spacings up to eight times apart
            ax[a].periodic = t % 5 == 4 && a == (int)(rnd() * d);
            const bool tiny = ax[a].periodic && rnd() < 0.5;
            ax[a].n = tiny ? 5 + (int)(rnd() * 12) : (d == 2 ? 60 + (int)(rnd() * 120) : 24 + (int)(rnd() * 16));
            ax[a].lo = -rnd();
            span = std::min(span, (ax[a].n - 1) * ax[a].h);
        }
        const int q = 2 + (int)(rnd() * (d == 2 ? 7 : 5));
        // landing points spread over 1 to 12 (16) cells of the finest axis
        const double S = (0.5 + rnd() * (d == 2 ? 7.0 : 5.0)) * h / 2.0, D = S * S / (4.0 * dt);
        const double drift = rnd() < 0.3 ? 0.0 : (rnd() - 0.5) * 4.0 * h / dt;
        check(d, ax, drift, D, dt, q, ball, 0.3 * span, t & 1);
    }
    // a short periodic last axis beside one of wide footprints: an index wraps once
    for (int d = 2; d <= 3; ++d)
        for (int n = 5; n <= 16; ++n)
            for (int L : {6, 8, 11, 12, 15}) {
                if (d == 3 && L > 12) continue;
                const double h = 0.01, S = (L - 2.5) * h / 2.0 / 2.930637420257244, dt = 1e-3;
                const Axis1 ax[3] = {{0.0, h, 40, 0}, {0.0, d == 2 ? 16 * h : h, d == 2 ? n : 24, d == 2},
                                     {0.0, 16 * h, n, 1}};
                check(d, ax, 0.0, S * S / (4.0 * dt), dt, d == 2 ? 8 : 6, false, 0.0, n & 1);
            }
    printf("%lld plans, %lld separable nodes, %lld reads checked, %lld outside\n", plans, sep_nodes, checked, bad);
    return bad || sep_nodes < 100000 ? 1 : 0;
}
