// Prints what the backprojectors' launch rules say of the plans on its input, one request a line:
//   plan NAME kz box_rows box_cols atan_degree valid_voxels tiles_x tiles_y nz slices_per_pitch pitches runs
//   class NAME            -> shape split poly4
//   batch NAME NAME ...   -> shape split poly4 of each
//   adjoint NAME          -> parts, window (float sums), window (fixed point)
//   order tiles_x tiles_y layers least -> "ok" if every layer's order takes each tile once
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "../../paper_2201_02309_amd/csrc/bp_rules.hpp"

using namespace kats;
using namespace kats::bpdev;

static void print(const BpClass &c) { std::cout << c.shape << ' ' << c.split << ' ' << c.poly4 << ' '; }

int main() {
    std::map<std::string, KParams> plans;
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string what, name;
        in >> what;
        if (what == "plan") {
            KParams k{};
            in >> name >> k.bp_kz >> k.bp_box_rows >> k.bp_box_cols >> k.atan_deg >> k.n_valid >> k.bp_tiles_x >>
                k.bp_tiles_y >> k.nz >> k.ns >> k.n_pitches >> k.bp_runs;
            k.nx = k.bp_tiles_x * kT;
            k.ny = k.bp_tiles_y * kT;
            plans[name] = k;
            continue;
        }
        if (what == "class") {
            in >> name;
            print(kernel_class(plans.at(name)));
        } else if (what == "batch") {
            std::vector<KParams> ks;
            while (in >> name) ks.push_back(plans.at(name));
            for (const BpClass &c : batch_classes(ks.data(), (int)ks.size())) print(c);
        } else if (what == "adjoint") {
            in >> name;
            const KParams &k = plans.at(name);
            std::cout << bpT_parts(k) << ' ' << bpT_window(k, false) << ' ' << bpT_window(k, true);
        } else if (what == "order") {
            unsigned tx, ty, layers, least;
            in >> tx >> ty >> layers >> least;
            bool ok = true;
            for (unsigned z = 0; z < layers; ++z) {
                std::vector<int> taken(tx * ty);
                for (unsigned l = 0; l < tx * ty; ++l) {
                    const TileAt t = xcd_tile(least, (int)tx, (int)ty, l, z, tx * ty * z);
                    if (t.x < 0 || t.y < 0 || t.x >= (int)tx || t.y >= (int)ty) ok = false;
                    else taken[(unsigned)t.y * tx + (unsigned)t.x]++;
                }
                for (int n : taken) ok = ok && n == 1;
            }
            std::cout << (ok ? "ok" : "wrong");
        }
        std::cout << '\n';
    }
    return 0;
}
